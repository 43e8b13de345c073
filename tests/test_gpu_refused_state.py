"""A refused state changes nothing: after any number of steps (the running
state is in either buffer) the run goes on bit for bit from where it was, and
its health bits stay; so too through device buffers and in a batch."""
import numpy as np
import pytest

from gpu_util import SCHEME_KW
from swe_inputs import river_channel

pytestmark = pytest.mark.gpu


def _problem(precision):
    from paper_2307_16758_amd.problem import prepare_scenario
    sc = river_channel(Lx=400.0, Ly=80.0, nx=37, ny=9, seed=5, inflow_q=15.0)
    pr = prepare_scenario(sc)
    l2g = pr.sub.l2g
    dt = np.float64 if precision else np.float32
    h = sc.h[l2g] * (1 + 0.1 * np.sin(np.arange(l2g.size)))
    return pr.mesh, [a.astype(dt) for a in (h, 0.2 * h, -0.1 * h)]


def _solver(mesh, precision, batch=1, name="muscl_minmod_rk2"):
    from paper_2307_16758_amd import swe
    s = swe.Solver(**SCHEME_KW[name], precision=precision)
    s.mesh_upload(mesh) if batch == 1 else s.mesh_upload_batch([mesh] * batch)
    return s


def _refuse(s, U, device):
    from paper_2307_16758_amd import swe
    for k, v in ((0, -1.0), (1, np.nan), (2, np.inf)):
        bad = [0.5 * u for u in U]
        bad[k][-1] = v
        if device:
            import torch
            bad = [torch.from_numpy(u).cuda() for u in bad]
            torch.cuda.synchronize()
        with pytest.raises(swe.SweError):
            s.set_state(*bad, t=7.0)


@pytest.mark.parametrize("steps", [0, 1, 2, 6])
@pytest.mark.parametrize("precision,batch,device", [(0, 1, False), (1, 1, True), (0, 3, True)])
def test_run_goes_on(precision, batch, device, steps):
    mesh, U = _problem(precision)
    U = [np.tile(u, batch) for u in U]
    a, b = (_solver(mesh, precision, batch) for _ in range(2))
    for s in (a, b):
        s.set_state(*U, t=1.0)
        s.step(steps)
    _refuse(b, U, device)
    for more in (0, 5):
        for s in (a, b):
            s.step(more)
        for x, y in zip(a.read_state(), b.read_state()):
            assert np.array_equal(x, y)
        assert a.time() == b.time() and a.local_dt() == b.local_dt()
    b.set_state(*U, t=2.0)          # an accepted one starts over
    assert b.time() == 2.0
    for x, y in zip(U, b.read_state()):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("steps", [1, 2])
def test_health_bits_stay(steps):
    """A step far too long leaves its mark; a refused state does not take it
    away, an accepted one does."""
    mesh, U = _problem(0)
    s = _solver(mesh, 0, name="hllc1")
    s.set_state(*U)
    s.step(steps, 60.0)
    bits = s.health()
    assert bits != 0
    _refuse(s, U, False)
    assert s.health() == bits
    s.set_state(*U)
    assert s.health() == 0


def test_refused_first_state():
    """Nothing was going on: there is still no state."""
    from paper_2307_16758_amd import swe
    mesh, U = _problem(0)
    s = _solver(mesh, 0)
    _refuse(s, U, False)
    with pytest.raises(swe.SweError):
        s.step(1)
    s.set_state(*U)
    s.step(1)
    s.sync()
