"""The network inside the first stage on meshes of one tile and a little more,
in every launch shape the autotuner runs, among them a thread per cell with
more edges than threads, where a wave is filled up past the tile's edges: the
bits of the network in a kernel of its own.  (Those lanes once read up to 256
bytes past the plan's memory in FP64, unused: 80 places of 32 bytes, read to
place 128, before 1280 bytes of central weights.)"""
import numpy as np
import pytest

from swe_inputs import river_channel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(6, 4), (5, 5), (9, 3), (13, 2), (8, 4), (17, 6)])
@pytest.mark.parametrize("precision", [0, 1])
def test_waves_filled_up(precision, nx, ny):
    from paper_2307_16758_amd import swe
    from paper_2307_16758_amd.limiter_train import init_params
    from paper_2307_16758_amd.problem import prepare_scenario
    sc = river_channel(Lx=10.0 * nx, Ly=10.0 * ny, nx=nx, ny=ny, seed=3, inflow_q=5.0)
    pr = prepare_scenario(sc)
    l2g = pr.sub.l2g
    h = 1.0 + sc.h[l2g] * (1 + 0.1 * np.sin(np.arange(l2g.size)))
    ref = None
    for in_stage in (0, 1):
        s = swe.Solver(precision=precision, scheme=1, integrator=1, limiter=3, phi_in_stage=in_stage)
        s.mesh_upload(pr.mesh)
        s.limiter_set_weights(init_params(4))
        s.set_state(h, 0.3 * h, 0.1 * h)
        if in_stage:
            s.autotune(2)
        s.step(9)
        out = s.read_state()
        s.close()
        if ref is None:
            ref = out
        for a, b in zip(ref, out):
            assert np.array_equal(a, b)
