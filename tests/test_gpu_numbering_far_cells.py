"""Numberings with some locality, whose halos are over the bound of Morton
ordered meshes: rows of the grid, and one cell in ten far away.  Tiles of 128
and 256 cells take them with a looser bound (the network inside an FP64 stage
does not at 256); WAF, the learned limiter in both places and batches too have
cell by cell the bits of the Morton-ordered run."""
import dataclasses

import numpy as np
import pytest

from gpu_util import SCHEME_KW
from swe_inputs import river_channel

pytestmark = pytest.mark.gpu

LEARNED = dict(scheme=1, integrator=1, limiter=3)
KW = {"hllc1": SCHEME_KW["hllc1"], "muscl": SCHEME_KW["muscl_superbee_rk2"], "waf": SCHEME_KW["waf"],
      "learned": dict(LEARNED), "learned_every": dict(LEARNED, phi_every=2),
      "network": dict(LEARNED, phi_in_stage=1)}


def _run(meshes, U, kw, steps, **cfg):
    from paper_2307_16758_amd import swe
    from paper_2307_16758_amd.limiter_train import init_params
    s = swe.Solver(**kw, **cfg)
    s.mesh_upload(meshes[0]) if len(meshes) == 1 else s.mesh_upload_batch(meshes)
    if kw["limiter"] == 3:
        s.limiter_set_weights(init_params(6))
    s.set_state(*U)
    s.step(steps)
    out = s.read_state() + (s.time(),)
    s.close()
    return out


def _renumbered(mesh, U, perm):
    inv = np.empty_like(perm)
    inv[perm] = np.arange(perm.size)
    nbr = mesh.cell_nbr.reshape(-1, 3)[perm]
    m = dataclasses.replace(
        mesh, cell_nodes=mesh.cell_nodes.reshape(-1, 3)[perm], cell_gid=mesh.cell_gid[perm],
        cell_nbr=np.where(nbr >= 0, inv[np.maximum(nbr, 0)], nbr).astype(np.int32),
        cell_b=mesh.cell_b[perm], cell_manning=mesh.cell_manning[perm])
    return m, [u[perm] for u in U]


def _problem(nx, ny, precision, seed=7):
    from paper_2307_16758_amd.problem import prepare_scenario
    sc = river_channel(Lx=2000.0, Ly=500.0, nx=nx, ny=ny, seed=seed, inflow_q=20.0)
    pr = prepare_scenario(sc)
    l2g = pr.sub.l2g
    dt = np.float64 if precision else np.float32
    h = sc.h[l2g] * (1.0 + 0.05 * np.sin(0.05 * sc.mesh.centroids()[l2g, 0]))
    return pr.mesh, [a.astype(dt) for a in (h, 0.3 * h, 0.1 * h)], l2g


def _orders(n, l2g, rng):
    far = np.arange(n)
    some = np.sort(rng.choice(n, n // 10, replace=False))
    far[some] = rng.permutation(some)
    return {"rows": np.argsort(l2g), "far": far, "random": rng.permutation(n)}


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", sorted(KW))
def test_far_cells(name, precision):
    kw = dict(KW[name], precision=precision)
    mesh, U, l2g = _problem(201, 51, precision)
    ref = _run([mesh], U, kw, 9)
    for order, perm in _orders(l2g.size, l2g, np.random.default_rng(3)).items():
        m, V = _renumbered(mesh, U, perm)
        for block in (0, 128, 256, 512):
            got = _run([m], V, kw, 9, block=block)
            for a, b in zip(ref[:3], got[:3]):
                assert np.array_equal(a[perm], b), (order, block)
            assert got[3] == ref[3], (order, block)


@pytest.mark.parametrize("name,precision", [("hllc1", 0), ("muscl", 1), ("waf", 0), ("waf", 1), ("learned", 0),
                                            ("network", 0)])
def test_batch_with_mixed_tiles(name, precision):
    """Scenarios of sizes that no tile ends with, far cells in each: tiles that
    hold two or three scenarios, and each one's own run."""
    kw = dict(KW[name], precision=precision)
    meshes, states, alone = [], [], []
    for i, (nx, ny) in enumerate(((41, 9), (7, 3), (5, 2), (97, 33))):
        mesh, U, l2g = _problem(nx, ny, precision, seed=11 + i)
        perm = _orders(l2g.size, l2g, np.random.default_rng(i))["far"]
        m, V = _renumbered(mesh, U, perm)
        meshes.append(m)
        states.append(V)
        alone.append(_run([m], V, kw, 7))
    for block in (0, 64, 256):
        got = _run(meshes, [np.concatenate(x) for x in zip(*states)], kw, 7, block=block)
        at = 0
        for ref in alone:
            n = ref[0].size
            for a, b in zip(ref[:3], got[:3]):
                assert np.array_equal(a, b[at:at + n]), block
            at += n
