"""The tile plan of the tiled stage kernel: any numbering of the cells and
any launch shape gives, cell by cell, the bits of the Morton-ordered run in
its default shape (which other tests compare with the oracle)."""
import numpy as np
import pytest

from gpu_util import SCHEME_KW
from swe_inputs import river_channel

pytestmark = pytest.mark.gpu


def _run(mesh, U, kw, steps, **cfg):
    from paper_2307_16758_amd import swe
    s = swe.Solver(**kw, **cfg)
    s.mesh_upload(mesh)
    s.set_state(*U)
    s.step(steps)
    out = s.read_state() + (s.time(),)
    s.close()
    return out


def _renumbered(mesh, U, perm):
    import dataclasses
    inv = np.empty_like(perm)
    inv[perm] = np.arange(perm.size)
    nbr = mesh.cell_nbr.reshape(-1, 3)[perm]
    m = dataclasses.replace(
        mesh, cell_nodes=mesh.cell_nodes.reshape(-1, 3)[perm], cell_gid=mesh.cell_gid[perm],
        cell_nbr=np.where(nbr >= 0, inv[np.maximum(nbr, 0)], nbr).astype(np.int32),
        cell_b=mesh.cell_b[perm], cell_manning=mesh.cell_manning[perm])
    return m, [u[perm] for u in U]


def _problem(nx, ny, precision):
    from paper_2307_16758_amd.problem import prepare_scenario
    sc = river_channel(Lx=500.0, Ly=100.0, nx=nx, ny=ny, seed=7, inflow_q=20.0)
    pr = prepare_scenario(sc)
    l2g = pr.sub.l2g
    dt = np.float64 if precision else np.float32
    x = sc.mesh.centroids()[l2g, 0]
    h = sc.h[l2g] * (1.0 + 0.05 * np.sin(0.05 * x))
    return pr.mesh, [a.astype(dt) for a in (h, 0.3 * h, 0.1 * h * np.cos(0.07 * x))]


# 31 x 2 cells: under one tile; 33 x 2 and 129 x 2: just over a tile and a
# ragged second one; 60 x 30: many tiles of every size
@pytest.mark.parametrize("nx,ny", [(31, 1), (33, 1), (43, 3), (60, 30)])
@pytest.mark.parametrize("name,precision", [("hllc1", 0), ("muscl_superbee_rk2", 0),
                                            ("muscl_vanalbada_rk2", 1)])
def test_numbering_without_locality(nx, ny, name, precision):
    """Random and row-reversed numberings: halos far over the bounds, so tiles
    are cut or smaller ones taken."""
    kw = dict(SCHEME_KW[name], precision=precision)
    mesh, U = _problem(nx, ny, precision)
    ref = _run(mesh, U, kw, 9)
    n = mesh.n_total
    rng = np.random.default_rng(5)
    jump = np.arange(n)
    jump[::97] = rng.permutation(jump[::97])          # a few far cells in many tiles
    for perm in (rng.permutation(n), np.arange(n)[::-1].copy(), jump):
        m, V = _renumbered(mesh, U, perm)
        for block in (0, 256):
            got = _run(m, V, kw, 9, block=block)
            for a, b in zip(ref[:3], got[:3]):
                assert np.array_equal(a[perm], b), block
            assert got[3] == ref[3]


@pytest.mark.parametrize("name,precision", [("hllc1", 1), ("muscl_minmod_rk2", 0), ("muscl_minmod_rk2", 1)])
def test_launch_shapes_agree_bitwise(name, precision):
    """Tiles of 64 to 512 cells, a thread per edge (the default of a small
    mesh) and, after the autotuner, whichever shape it chose."""
    from paper_2307_16758_amd import swe
    kw = dict(SCHEME_KW[name], precision=precision)
    mesh, U = _problem(90, 41, precision)
    ref = _run(mesh, U, kw, 13)
    for cfg in (dict(block=64), dict(block=128), dict(block=256), dict(block=512),
                dict(block=256, waves=6), dict(block=256, waves=7)):
        got = _run(mesh, U, kw, 13, **cfg)
        for a, b in zip(ref[:3], got[:3]):
            assert np.array_equal(a, b), cfg
        assert got[3] == ref[3]
    s = swe.Solver(**kw)
    s.mesh_upload(mesh)
    s.set_state(*U)
    s.autotune(4)
    s.step(13)
    for a, b in zip(ref[:3], s.read_state()):
        assert np.array_equal(a, b)
    s.close()


@pytest.mark.parametrize("name,precision", [("muscl_minmod_rk2", 0), ("waf", 0), ("hllc1", 1)])
def test_roughness_of_one_value_and_of_many(name, precision):
    """A scenario whose cells share one Manning n takes it from one place: the
    same bits as read cell by cell (one dry cell's value made to differ)."""
    import dataclasses
    kw = dict(SCHEME_KW[name], precision=precision)
    mesh, U = _problem(60, 30, precision)
    assert np.all(mesh.cell_manning == mesh.cell_manning[0]) and mesh.cell_manning[0] > 0
    dry = int(np.argmax(mesh.cell_b))
    assert U[0][dry] == 0.0
    man = mesh.cell_manning.copy()
    man[dry] *= 2.0
    ref = _run(mesh, U, kw, 20)
    got = _run(dataclasses.replace(mesh, cell_manning=man), U, kw, 20)
    assert ref[0][dry] == 0.0                          # it stayed dry: its n was never used
    for a, b in zip(ref[:3], got[:3]):
        assert np.array_equal(a, b)
    assert got[3] == ref[3]


def test_mesh_beyond_the_cache_equals_its_small_tiles():
    """2.8 million cells (a step's arrays over the bound) load their geometry
    as a stream in 256-cell tiles; tiles of 512 cells do not: same bits."""
    from paper_2307_16758_amd.problem import prepare_scenario
    sc = river_channel(nx=2650, ny=530, seed=9)
    pr = prepare_scenario(sc)
    l2g = pr.sub.l2g
    h = (sc.h[l2g] * (1 + 0.02 * np.sin(0.01 * np.arange(l2g.size)))).astype(np.float32)
    U = [h, 0.3 * h, 0.1 * h]
    kw = dict(SCHEME_KW["muscl_minmod_rk2"], precision=0)
    ref = _run(pr.mesh, U, kw, 4)
    got = _run(pr.mesh, U, kw, 4, block=512)
    for a, b in zip(ref[:3], got[:3]):
        assert np.array_equal(a, b)
