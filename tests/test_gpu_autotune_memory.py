"""The autotuner where memory is short: a shape whose plan cannot be had is
left out (only the run's state and clock have to be saved), no more than one
plan is held beside the running and the fastest shape's, and in every case the
run goes on with the same bits."""
import ctypes as C

import numpy as np
import pytest

from gpu_util import SCHEME_KW
from swe_inputs import river_channel

pytestmark = pytest.mark.gpu


class Pool:
    """Allocator callbacks of a context with a budget of bytes."""

    def __init__(self):
        from paper_2307_16758_amd import swe
        self.hip, self.live, self.left = swe.lib(), {}, None
        self.peak = 0
        self.kw = dict(alloc=swe.ALLOC_FN(self._alloc), free=swe.FREE_FN(self._free))

    def _alloc(self, nbytes, user):
        if self.left is not None and nbytes > self.left:
            return None
        p = C.c_void_p()
        if self.hip.hipMalloc(C.byref(p), C.c_size_t(nbytes)) != 0:
            return None
        if self.left is not None:
            self.left -= nbytes
        self.live[p.value] = nbytes
        self.peak = max(self.peak, len(self.live))
        return p.value

    def _free(self, p, user):
        n = self.live.pop(p)
        if self.left is not None:
            self.left += n
        self.hip.hipFree(C.c_void_p(p))


def _run(nx, ny, name, precision, pool):
    from paper_2307_16758_amd import swe
    from paper_2307_16758_amd.problem import prepare_scenario
    sc = river_channel(Lx=500.0, Ly=100.0, nx=nx, ny=ny, seed=7, inflow_q=20.0)
    pr = prepare_scenario(sc)
    l2g = pr.sub.l2g
    h = sc.h[l2g] * (1 + 0.05 * np.sin(np.arange(l2g.size)))
    s = swe.Solver(**SCHEME_KW[name], precision=precision, **(pool.kw if pool else {}))
    s.mesh_upload(pr.mesh)
    s.set_state(h, 0.2 * h, -0.1 * h)
    s.step(3)
    return s, l2g.size


# one launch per step, tiles of 64, 128 and 256 cells by size
CASES = [(90, 41, "muscl_minmod_rk2", 0), (90, 41, "hllc1", 0), (370, 150, "muscl_minmod_rk2", 0),
         (370, 150, "waf", 1), (500, 260, "muscl_minmod_rk2", 0)]


@pytest.mark.parametrize("nx,ny,name,precision", CASES)
def test_no_memory_for_other_plans(nx, ny, name, precision):
    twin, _ = _run(nx, ny, name, precision, None)
    pool = Pool()
    s, n = _run(nx, ny, name, precision, pool)
    held = dict(pool.live)
    clock = 4 * 17 * 16 * 8                                 # slots, lines, words, bytes
    pool.left = 4 * (8 if precision else 4) * n + clock     # the save buffers and no more
    s.autotune(3)
    assert pool.live == held
    for x in (s, twin):
        x.step(13)
    for a, b in zip(s.read_state(), twin.read_state()):
        assert np.array_equal(a, b)
    assert s.time() == twin.time()
    s.close()
    assert not pool.live


@pytest.mark.parametrize("nx,ny,name,precision", CASES)
def test_plans_held(nx, ny, name, precision):
    twin, _ = _run(nx, ny, name, precision, None)
    pool = Pool()
    s, _ = _run(nx, ny, name, precision, pool)
    held = len(pool.live)
    pool.peak = held
    s.autotune(3)
    # two save buffers, the fastest shape's plan and the one being tried
    assert pool.peak <= held + 4
    assert len(pool.live) <= held
    for x in (s, twin):
        x.step(13)
    for a, b in zip(s.read_state(), twin.read_state()):
        assert np.array_equal(a, b)
    s.close()
    assert not pool.live
