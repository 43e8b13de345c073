"""Half-edges without an upwind cell (a cell with two boundary edges) stay
first order: on a mesh of separate squares of two triangles each, where every
interior edge is such a one, every MUSCL run gives the bits of first-order
HLLC, on wet cells of a sloping bed too (eta - h is not b there)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

MINMOD, SUPERBEE, VANALBADA, LEARNED, ZEROSLOPE = range(5)


def _squares(n, precision):
    """n unit squares apart from each other, walls all around, random beds and
    states; every ninth cell dry."""
    from paper_2307_16758_amd import swe
    rng = np.random.default_rng(n)
    x = 2.0 * np.arange(n)
    xy = np.stack([np.stack([x, x + 1, x + 1, x], 1), np.tile([0.0, 0.0, 1.0, 1.0], (n, 1))], 2).reshape(-1, 2)
    q = 4 * np.arange(n)[:, None]
    tri = np.concatenate([q + [0, 1, 2], q + [0, 2, 3]], 1).reshape(-1, 3)
    nbr = np.full((n, 2, 3), -1, np.int32)
    nbr[:, 0, 2] = 2 * np.arange(n) + 1
    nbr[:, 1, 0] = 2 * np.arange(n)
    none = np.zeros(0, np.int32)
    m = swe.MeshArrays(node_xy=xy, n_owned=2 * n, cell_nodes=tri.astype(np.int32),
                       cell_gid=rng.permutation(2 * n).astype(np.int64), cell_nbr=nbr.reshape(-1, 3),
                       cell_b=rng.uniform(-4.0, 6.0, 2 * n), cell_manning=np.full(2 * n, 0.03),
                       peers=none, recv_off=np.zeros(1, np.int32), send_off=np.zeros(1, np.int32), send_idx=none)
    h = rng.uniform(0.2, 3.0, 2 * n)
    h[::9] = 0.0
    dt = np.float64 if precision else np.float32
    return m, [a.astype(dt) for a in (h, h * rng.normal(size=2 * n), h * rng.normal(size=2 * n))]


@pytest.mark.parametrize("n", [1, 40, 700])
@pytest.mark.parametrize("limiter", [MINMOD, SUPERBEE, VANALBADA, LEARNED, ZEROSLOPE])
@pytest.mark.parametrize("integrator", [0, 1])
@pytest.mark.parametrize("precision", [0, 1])
def test_no_upwind_cell_is_first_order(precision, integrator, limiter, n):
    from paper_2307_16758_amd import swe
    from paper_2307_16758_amd.limiter_train import init_params
    mesh, U = _squares(n, precision)

    def run(**cfg):
        s = swe.Solver(precision=precision, integrator=integrator, **cfg)
        s.mesh_upload(mesh)
        if cfg.get("limiter") == LEARNED:
            s.limiter_set_weights(init_params(2))
        s.set_state(*U)
        s.step(5, 0.002)
        out = s.read_state()
        s.close()
        return out

    ref = run(scheme=swe.HLLC1)
    for more in (dict(), dict(block=128), dict(phi_in_stage=1)):
        if "phi_in_stage" in more and limiter != LEARNED:
            continue
        for a, b in zip(ref, run(scheme=swe.MUSCL, limiter=limiter, **more)):
            assert np.array_equal(a, b), more
