"""What the waiting calls return right behind queued steps (of the tiled and of
the one-thread-per-cell kernel, alone and in a batch, on a borrowed stream that
is busy): the values of a run that was waited for first."""
import numpy as np
import pytest

from gpu_util import SCHEME_KW
from swe_inputs import river_channel

pytestmark = pytest.mark.gpu


def _solver(kw, batch, precision, **more):
    from paper_2307_16758_amd import swe
    from paper_2307_16758_amd.problem import prepare_scenario
    sc = river_channel(Lx=400.0, Ly=80.0, nx=37, ny=9, seed=5, inflow_q=15.0)
    pr = prepare_scenario(sc)
    s = swe.Solver(**kw, precision=precision, **more)
    s.mesh_upload(pr.mesh) if batch == 1 else s.mesh_upload_batch([pr.mesh] * batch)
    h = np.tile(sc.h[pr.sub.l2g], batch)
    s.set_state(h, 0.2 * h, -0.1 * h, t=0.5)
    return s


CALLS = ["sync", "time", "local_dt", "health", "last_step_ms"]


@pytest.mark.parametrize("cell_kernel", [0, 1])
@pytest.mark.parametrize("batch,precision,call", [(b, p, c) for b, p in ((1, 0), (3, 1), (70, 0))
                                                  for c in CALLS + ["scenario_times"] * (b > 1)])
def test_values_behind_queued_steps(batch, precision, cell_kernel, call):
    import torch
    kw = dict(SCHEME_KW["muscl_minmod_rk2"], cell_kernel=cell_kernel)
    st = torch.cuda.Stream()
    s, twin = _solver(kw, batch, precision, stream=st), _solver(kw, batch, precision)
    a = torch.randn(2048, 2048, device="cuda")
    torch.cuda.synchronize()
    for steps in (1, 7):
        twin.step(steps)
        torch.cuda.synchronize()
        with torch.cuda.stream(st):
            for _ in range(5):
                a = torch.tanh(a @ a)
        s.step(steps)
        got = getattr(s, call)()
        if call == "last_step_ms":
            assert got > 0.0
        else:
            ref = getattr(twin, call)()
            assert np.array_equal(got, ref) if got is not None else ref is None
    assert s.time() == twin.time() > 0.5
