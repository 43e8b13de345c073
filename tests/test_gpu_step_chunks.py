"""However a run is cut into calls (single steps, the short and the long
graph, a fixed step between), the state and the clock are the same bits."""
import numpy as np
import pytest

from gpu_util import SCHEME_KW
from swe_inputs import river_channel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,more", [("hllc1", {}), ("muscl_minmod_rk2", {}), ("waf", {}),
                                       ("muscl_minmod_rk2", dict(limiter=3, phi_every=3))])
def test_calls_of_any_length(name, more):
    from paper_2307_16758_amd import swe
    from paper_2307_16758_amd.limiter_train import init_params
    from paper_2307_16758_amd.problem import prepare_scenario
    sc = river_channel(Lx=400.0, Ly=80.0, nx=41, ny=9, seed=6, inflow_q=15.0)
    pr = prepare_scenario(sc)
    l2g = pr.sub.l2g
    kw = dict(SCHEME_KW[name], precision=0, **{k: v for k, v in more.items() if k != "limiter"})
    kw["limiter"] = more.get("limiter", kw["limiter"])
    h = (sc.h[l2g] * (1 + 0.1 * np.sin(np.arange(l2g.size)))).astype(np.float32)
    ref = None
    for calls in ([1] * 109, [109], [48, 61], [5, 49, 55], [6, 24, 30, 49], [53, 56]):
        assert sum(calls) == 109
        s = swe.Solver(**kw)
        s.mesh_upload(pr.mesh)
        if kw["limiter"] == 3:
            s.limiter_set_weights(init_params(1))
        s.set_state(h, 0.2 * h, -0.1 * h)
        if calls == [109]:
            s.prepare()
        for k in calls:
            s.step(k)
        out = s.read_state() + (s.time(),)
        s.close()
        if ref is None:
            ref = out
        for a, b in zip(ref[:3], out[:3]):
            assert np.array_equal(a, b), calls
        assert out[3] == ref[3]
