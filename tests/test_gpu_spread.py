"""Spread relaxation (several workgroups per RVE) against the incidence kernel,
whose arithmetic it shares: states and iteration counts agree bit for bit, the
norms (summed in another order) to rounding."""
import re

import numpy as np
import pytest

from gpu_common import require_gpu
from paper_2306_09427_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rb():
    return require_gpu()


@pytest.fixture(scope="module")
def nets():
    # 4 parts, partly filled; 8 parts; every node of degree 6 (two extra records each)
    return [synth.voronoi_network(1000, [41, 0, 0]), synth.voronoi_network(2000, [41, 1, 0]), synth.lattice_network(15)]


def run(rb, nets, engine, F, spin=None, warm=None, **kw):
    o = dict(precision=rb.MIXED, alpha=0.5, c=0.3, tol_abs=0.0, tol_rel=1e-6, n_max=4000, check_every=1, engine=engine)
    o.update(kw)
    b = rb.Batch(synth.pack(nets), **o)
    if engine == rb.ENGINE_AUTO:
        assert all(re.match(r"incidence\((global,)?\d+(-\d+)?x\d+\):", g) for g in b.describe().split(";")[:-1]), b.describe()
    if spin is not None:
        b.team_spin_limit(spin)
    out = []
    for f in [F] + ([warm] if warm is not None else []):
        if out:
            b.set_opts(init=rb.INIT_WARM, **o)
        sig, st, stats = b.solve(f, stats=True)
        out.append((sig, st, stats, b.export_state()[1]))
    b.close()
    return out


def same(x, y):
    for (s0, t0, q0, h0), (s1, t1, q1, h1) in zip(x, y):
        assert np.array_equal(t0, t1) and np.array_equal(q0["iters"], q1["iters"])
        assert np.array_equal(h0, h1) and np.array_equal(s0, s1, equal_nan=True)
        for k in ("R", "D", "Fb"):
            np.testing.assert_allclose(q0[k], q1[k], rtol=1e-11, atol=0)


def stretch(n, e=0.1):
    F = np.broadcast_to(np.diag([1 + e, 1 - e / 3, 1 - e / 3]), (n, 3, 3)).copy()
    F[:, 0, 1] = 0.02 * np.arange(n) / max(n, 1)
    return F


@pytest.mark.parametrize("opt", ["lumped", "scaled", "linear", "late", "n_max"])
def test_bitwise_against_incidence(rb, nets, opt):
    kw = dict(lumped={}, scaled=dict(mass=rb.MASS_SCALED), linear=dict(law=rb.LAW_LINEAR), late=dict(check_every=7),
              n_max=dict(n_max=50, check_every=8))[opt]
    F, W = stretch(3), stretch(3, 0.12)
    same(run(rb, nets, rb.ENGINE_AUTO, F, warm=W, **kw), run(rb, nets, rb.ENGINE_INCIDENCE, F, warm=W, **kw))


def test_more_rves_than_teams_and_bad_F(rb, nets):
    many = [nets[0]] * 70 + [nets[2]] * 35
    F = stretch(len(many))
    F[3] = np.diag([-1.0, 1.0, 1.0])
    F[101, 0, 0] = np.nan
    kw = dict(n_max=300, check_every=10)
    x, y = run(rb, many, rb.ENGINE_AUTO, F, **kw), run(rb, many, rb.ENGINE_INCIDENCE, F, **kw)
    assert (x[0][1][[3, 101]] == rb.ST_BAD_F).all()
    same(x, y)


def test_teams_that_give_up(rb, nets):
    """One poll per word: the incidence kernel behind takes what the teams left."""
    F = stretch(3)
    same(run(rb, nets, rb.ENGINE_AUTO, F, spin=1), run(rb, nets, rb.ENGINE_INCIDENCE, F))


@pytest.mark.parametrize("spin", [None, 1])
def test_spread_tangent_and_vjp(rb, nets, spin):
    """Tangent columns and VJPs over several workgroups against the streamed
    kernel at the same states (one of them not converged, and the lattice's
    stiffness indefinite under the lateral compression); spin 1: the teams
    give up and the streamed kernel behind takes their tasks."""
    some = [nets[0], nets[2], nets[0], nets[1]]
    o = dict(precision=rb.MIXED, mass=rb.MASS_SCALED, alpha=0.5, c=0.1, tol_abs=0.0, tol_rel=1e-5, n_max=20000,
             check_every=8, cg_tol=1e-9)
    b = rb.Batch(synth.pack(some), **o)
    F, h, st = (b.solve(stretch(4)), b.export_state())[1]
    assert (st == 0).all()
    st[2] = 1
    g = np.random.default_rng(3).standard_normal((4, 3, 3))
    out = []
    for engine in (rb.ENGINE_AUTO, rb.ENGINE_STREAMED):
        b.set_opts(engine=engine, **o)
        if spin is not None:
            b.team_spin_limit(spin)
        b.import_state(F, h, st)
        C, cs = b.tangent()
        C2, _ = b.tangent()
        gF, gs = b.vjp(g)
        assert np.array_equal(C, C2, equal_nan=True)
        assert cs.tolist() == [0, rb.ST_CG_INDEFINITE, rb.ST_NO_STATE, 0] and gs[[0, 2, 3]].tolist() == [0, rb.ST_NO_STATE, 0]
        out.append((C, gF))
    b.close()
    on = [0, 3]
    scale = np.abs(out[1][0][on]).max(axis=(1, 2))
    assert np.isnan(out[0][0][2]).all() and np.isnan(out[0][1][2]).all()
    assert np.all(np.abs(out[0][0] - out[1][0])[on].max(axis=(1, 2)) < 1e-7 * scale)
    assert np.all(np.abs(out[0][1] - out[1][1])[on].max(axis=(1, 2)) < 1e-7 * scale * np.abs(g).max() * 9)
