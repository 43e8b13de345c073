"""The launch shapes that the size rule takes on large meshes: a thread per
cell in tiles of 256 cells, and geometry loaded as a stream.  The bits are
those of a thread per edge (a small mesh alone, the parts of a large one) and
of smaller tiles without the stream."""
import numpy as np
import pytest

from gpu_util import SCHEME_KW
from swe_inputs import river_channel

pytestmark = pytest.mark.gpu

LEARNED = dict(scheme=1, integrator=1, limiter=3)
KW = {"hllc1": SCHEME_KW["hllc1"], "superbee": SCHEME_KW["muscl_superbee_rk2"],
      "vanalbada": SCHEME_KW["muscl_vanalbada_rk2"], "euler": SCHEME_KW["muscl_minmod_euler"],
      "waf": SCHEME_KW["waf"], "learned": LEARNED, "network": dict(LEARNED, phi_in_stage=1)}


def _state(sc, l2g, precision):
    dt = np.float64 if precision else np.float32
    h = sc.h[l2g] * (1.0 + 0.05 * np.sin(0.05 * sc.mesh.centroids()[l2g, 0]))
    return [a.astype(dt) for a in (h, 0.3 * h, 0.1 * h)]


def _run(meshes, U, kw, steps, dt=0.0, **cfg):
    from paper_2307_16758_amd import swe
    from paper_2307_16758_amd.limiter_train import init_params
    s = swe.Solver(**kw, **cfg)
    s.mesh_upload(meshes[0]) if len(meshes) == 1 else s.mesh_upload_batch(meshes)
    if kw["limiter"] == 3:
        s.limiter_set_weights(init_params(6))
    s.set_state(*U)
    s.step(steps, dt)
    out = s.read_state()
    s.close()
    return out


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", sorted(KW))
def test_a_thread_per_cell_or_per_edge(name, precision):
    """7,380 cells alone take a thread per edge (or one launch per step), 32
    copies of them in a batch, 236,160 cells, a thread per cell; most tiles of
    the batch lie across two copies, or within one."""
    from paper_2307_16758_amd.problem import prepare_scenario
    kw = dict(KW[name], precision=precision)
    sc = river_channel(Lx=500.0, Ly=100.0, nx=90, ny=41, seed=7, inflow_q=20.0)
    pr = prepare_scenario(sc)
    U = _state(sc, pr.sub.l2g, precision)
    ref = _run([pr.mesh], U, kw, 7)
    n = U[0].size
    for block in (0, 64, 128):
        got = _run([pr.mesh] * 32, [np.tile(u, 32) for u in U], kw, 7, block=block)
        for a, b in zip(ref, got):
            assert np.array_equal(np.tile(a, 32), b), block


@pytest.mark.parametrize("name,precision", [("hllc1", 0), ("superbee", 0), ("waf", 0), ("learned", 0),
                                            ("network", 0), ("superbee", 1), ("waf", 1), ("learned", 1)])
def test_large_mesh_and_its_parts(name, precision):
    """240,000 cells FP32, 140,000 FP64 (a thread per cell), and one step of
    their halves (a thread per edge) on the cells these own."""
    from paper_2307_16758_amd.problem import prepare_scenario
    kw = dict(KW[name], precision=precision)
    nx, ny = (500, 140) if precision else (750, 160)
    sc = river_channel(Lx=5000.0, Ly=1000.0, nx=nx, ny=ny, seed=5, inflow_q=200.0)
    pr = prepare_scenario(sc)
    whole = _run([pr.mesh], _state(sc, pr.sub.l2g, precision), kw, 1, 0.01)
    at = np.empty(sc.n_cells, np.int64)
    at[pr.sub.l2g] = np.arange(sc.n_cells)
    for p in range(2):
        q = prepare_scenario(sc, P=2, p=p, k=4)
        l2g, no = q.sub.l2g, q.sub.n_owned
        part = _run([q.mesh], _state(sc, l2g, precision), kw, 1, 0.01)
        for a, b in zip(whole, part):
            assert np.array_equal(a[at[l2g[:no]]], b[:no])


@pytest.fixture(scope="module")
def beyond_the_cache():
    from paper_2307_16758_amd.problem import prepare_scenario
    sc = river_channel(nx=2650, ny=530, seed=9)
    pr = prepare_scenario(sc)
    return pr.mesh, sc, pr.sub.l2g


@pytest.mark.parametrize("name,precision", [("hllc1", 1), ("superbee", 1), ("learned", 0), ("network", 0)])
def test_geometry_as_a_stream(beyond_the_cache, name, precision):
    """2.8 million cells: over the bound of a step's arrays in 256-cell tiles
    (the stream), which 128-cell tiles do not use."""
    mesh, sc, l2g = beyond_the_cache
    kw = dict(KW[name], precision=precision)
    U = _state(sc, l2g, precision)
    ref = _run([mesh], U, kw, 2)
    for a, b in zip(ref, _run([mesh], U, kw, 2, block=128)):
        assert np.array_equal(a, b)
