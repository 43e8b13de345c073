"""A MUSCL-RK2 step of a small mesh takes one launch (k_step_tiled): the same
bits as its two stage launches, on one tile, on ragged tiles and on both sides
of the size where the rule stops; a part with ghost rows keeps two."""
import numpy as np
import pytest

from gpu_util import SCHEME_KW

pytestmark = pytest.mark.gpu

LIMITERS = ["muscl_minmod_rk2", "muscl_superbee_rk2", "muscl_vanalbada_rk2", "zeroslope"]


def _kw(name, precision):
    kw = dict(SCHEME_KW[name]) if name in SCHEME_KW else dict(scheme=1, integrator=1, limiter=4)
    return dict(kw, precision=precision)


def _problem(nx, ny, precision, **part):
    from paper_2307_16758_amd.problem import prepare_scenario
    from swe_inputs import river_channel
    sc = river_channel(Lx=500.0, Ly=100.0, nx=nx, ny=ny, seed=7, inflow_q=20.0)
    pr = prepare_scenario(sc, **part)
    l2g = pr.sub.l2g
    x = sc.mesh.centroids()[l2g, 0]
    h = sc.h[l2g] * (1.0 + 0.05 * np.sin(0.05 * x))
    dt = np.float64 if precision else np.float32
    return pr, [a.astype(dt) for a in (h, 0.3 * h, 0.1 * h * np.cos(0.07 * x))]


def _run(pr, U, kw, steps, dt=0.0, series=None, **cfg):
    from paper_2307_16758_amd import swe
    s = swe.Solver(**kw, **cfg)
    s.mesh_upload(pr.mesh)
    if series:
        s.set_bc_series(*series)
    s.set_state(*U)
    kernel = s.step_kernel()
    s.step(steps, dt)
    out = s.read_state() + (s.time(), s.health())
    s.close()
    return kernel, out


def _same(a, b):
    for x, y in zip(a[:3], b[:3]):
        assert np.array_equal(np.asarray(x).view(np.uint8), np.asarray(y).view(np.uint8))
    assert a[3:] == b[3:]


@pytest.mark.parametrize("nx,ny", [(31, 1), (33, 1), (43, 3), (90, 41)])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", LIMITERS)
def test_one_launch_is_two(name, precision, nx, ny):
    pr, U = _problem(nx, ny, precision)
    kw = _kw(name, precision)
    # the second stage takes its inflow at the end of the step
    series = ([0.0, 0.3, 0.6, 5.0], [20.0, 90.0, 15.0, 60.0])
    for cfg in (dict(), dict(cfl_rule=1), dict(dt=0.02), dict(series=series)):
        k1, one = _run(pr, U, kw, 31, **cfg)
        k2, two = _run(pr, U, kw, 31, block=128, **cfg)
        assert k1 == ("k_step_tiled", 1) and k2 == ("k_stage_tiled", 2)
        _same(one, two)


@pytest.mark.parametrize("precision,most", [(0, 98304), (1, 49152)])
def test_sizes_around_the_rule(precision, most):
    """The largest mesh of one launch per step and the smallest of two."""
    ny = 64
    for nx, kernel in ((most // (2 * ny), ("k_step_tiled", 1)), (most // (2 * ny) + 1, ("k_stage_tiled", 2))):
        pr, U = _problem(nx, ny, precision)
        kw = _kw("muscl_superbee_rk2", precision)
        k, got = _run(pr, U, kw, 12)
        assert k == kernel
        _same(got, _run(pr, U, kw, 12, block=256)[1])


def test_part_keeps_two_launches():
    pr, U = _problem(90, 41, 0, P=3, p=1, k=4)
    assert pr.sub.n_total > pr.sub.n_owned
    kw = _kw("muscl_minmod_rk2", 0)
    kernel, got = _run(pr, U, kw, 4)
    assert kernel == ("k_stage_tiled", 2)
    _same(got, _run(pr, U, kw, 4, block=256)[1])
