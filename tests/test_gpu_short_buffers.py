"""Device buffers that end before n_total values are refused by swe_set_state
and swe_read_state (through the C ABI, which has pointers only), and the run
goes on; buffers that hold exactly n_total are taken."""
import ctypes as C

import numpy as np
import pytest

from gpu_util import SCHEME_KW
from swe_inputs import river_channel

pytestmark = pytest.mark.gpu

ERR_DEVICE = -6


@pytest.fixture
def hip_alloc():
    """hipMalloc of an exact size (a framework's allocator would give a part of
    a larger block)."""
    from paper_2307_16758_amd import swe
    hip = swe.lib()  # (the HIP runtime that the library is linked to)
    got = []

    def alloc(nbytes):
        p = C.c_void_p()
        assert hip.hipMalloc(C.byref(p), C.c_size_t(nbytes)) == 0
        got.append(p)
        return p
    yield alloc
    for p in got:
        hip.hipFree(p)


@pytest.mark.parametrize("precision", [0, 1])
def test_short_device_buffers(hip_alloc, precision):
    from paper_2307_16758_amd import swe
    from paper_2307_16758_amd.problem import prepare_scenario
    sc = river_channel(Lx=400.0, Ly=80.0, nx=37, ny=9, seed=5, inflow_q=15.0)
    pr = prepare_scenario(sc)
    l2g = pr.sub.l2g
    L, n, ts = swe.lib(), l2g.size, 8 if precision else 4
    # one value short, within the last page of the allocation
    assert (n * ts - ts) % 4096 != 0
    s, twin = (swe.Solver(**SCHEME_KW["muscl_minmod_rk2"], precision=precision) for _ in range(2))
    h = sc.h[l2g] * (1 + 0.1 * np.sin(np.arange(n)))
    for x in (s, twin):
        x.mesh_upload(pr.mesh)
        x.set_state(h, 0.2 * h, -0.1 * h)
        x.step(2)
    full = [hip_alloc(n * ts) for _ in range(3)]
    short = hip_alloc(n * ts - ts)
    assert L.swe_read_state(s.ctx, *full, swe.DEVICE) == 0
    for k in range(3):
        bufs = full[:k] + [short] + full[k + 1:]
        assert L.swe_set_state(s.ctx, *bufs, swe.DEVICE, C.c_double(3.0)) == ERR_DEVICE
        assert L.swe_read_state(s.ctx, *bufs, swe.DEVICE) == ERR_DEVICE
        # the same buffer, from its second value on
        bufs[k] = C.c_void_p(full[k].value + ts)
        assert L.swe_set_state(s.ctx, *bufs, swe.DEVICE, C.c_double(3.0)) == ERR_DEVICE
    for x in (s, twin):
        x.step(3)
    for a, b in zip(s.read_state(), twin.read_state()):
        assert np.array_equal(a, b)
    assert s.time() == twin.time()
    # `full` still holds the state after two steps
    assert L.swe_set_state(s.ctx, *full, swe.DEVICE, C.c_double(0.0)) == 0
    s.step(1)
    s.sync()
