"""Paths of the relaxation and the tangent over several workgroups per RVE that a single
ordinary call does not take: teams that give up in a warm start, exchange areas handed from
one RVE to the next, a captured graph, two batches whose teams compete for the CUs."""
import threading

import numpy as np
import pytest

from gpu_common import require_gpu
from paper_2306_09427_amd import synth
from test_gpu_spread import run, same, stretch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rb():
    return require_gpu()


@pytest.fixture(scope="module")
def net1000():
    return synth.voronoi_network(1000, [41, 0, 0])


@pytest.mark.parametrize("n_max", [1, 8])
def test_warm_start_with_teams_that_give_up(rb, net1000, n_max):
    """Few polls per word: some members give up at the last exchange, when others have
    stored their part of the result.  The kernel behind starts from the caller's state."""
    nets, W = [net1000] * 84, stretch(84, 0.12)
    o = dict(precision=rb.MIXED, alpha=0.5, c=0.3, tol_abs=0.0, tol_rel=1e-12, n_max=n_max, check_every=1)
    b0 = rb.Batch(synth.pack(nets), engine=rb.ENGINE_INCIDENCE, **o)
    b0.solve(stretch(84))
    start = b0.export_state()
    b = rb.Batch(synth.pack(nets), **o)
    out = []
    for batch, spins in ((b0, [None]), (b, [2, 3, 4, 5] * 3)):
        batch.set_opts(init=rb.INIT_WARM, engine=rb.ENGINE_INCIDENCE if batch is b0 else rb.ENGINE_AUTO, **o)
        for spin in spins:
            if spin:
                batch.team_spin_limit(spin)
            batch.import_state(*start)
            sig, st, stats = batch.solve(W, stats=True)
            assert (st == rb.ST_MAXITER).all()
            out.append([(sig, st, stats, batch.export_state()[1])])
        batch.close()
    for x in out[1:]:
        same(x, out[0])


@pytest.fixture(scope="module")
def mixed_sizes(net1000):
    """More RVEs than exchange areas: 4000 seeds make the areas large (12 parts or more),
    and the smaller networks take them over with 2 and 3 parts."""
    return [synth.voronoi_network(4000, [41, 9, 0])] + [net1000] * 40 + [synth.voronoi_network(650, [41, 6, 0])] * 270


def test_areas_handed_on(rb, mixed_sizes):
    F = stretch(len(mixed_sizes))
    F[[5, 300]] = np.diag([-1.0, 1.0, 1.0])
    kw = dict(n_max=60, check_every=8)
    x, y = (run(rb, mixed_sizes, e, F, warm=1.01 * F, **kw) for e in (rb.ENGINE_AUTO, rb.ENGINE_INCIDENCE))
    assert (x[0][1][[5, 300]] == rb.ST_BAD_F).all()
    same(x, y)


def test_areas_handed_on_in_the_tangent(rb, mixed_sizes):
    """31 RVEs of nine columns and more tasks than areas; one RVE without a state."""
    some = mixed_sizes[:31]
    o = dict(precision=rb.MIXED, mass=rb.MASS_SCALED, alpha=0.5, c=0.1, tol_abs=0.0, tol_rel=1e-4, n_max=20000,
             check_every=8, cg_tol=1e-9)
    b = rb.Batch(synth.pack(some), **o)
    b.solve(stretch(31))
    F, h, st = b.export_state()
    assert (st == 0).all()
    st[4] = 1
    out = []
    for engine in (rb.ENGINE_AUTO, rb.ENGINE_STREAMED):
        b.set_opts(engine=engine, **o)
        b.import_state(F, h, st)
        out.append(b.tangent())
    b.close()
    (C, cs), (Cr, cr) = out
    assert np.array_equal(cs, cr) and cs[4] == rb.ST_NO_STATE and np.isnan(C[4]).all()
    on = np.flatnonzero(cs == 0)
    assert len(on) >= 25
    scale = np.abs(Cr[on]).max(axis=(1, 2))
    assert np.all(np.abs(C[on] - Cr[on]).max(axis=(1, 2)) < 1e-7 * scale)


def test_captured_graph(rb, net1000):
    import torch
    nets = [net1000, synth.voronoi_network(2000, [41, 1, 0]), synth.voronoi_network(60, [41, 5, 0])]
    b = rb.Batch(synth.pack(nets), precision=rb.MIXED, mass=rb.MASS_SCALED, alpha=0.5, c=0.1, tol_abs=0.0, tol_rel=1e-4,
                 n_max=20000, check_every=8)
    assert "x512)" in b.describe(), b.describe()
    s = torch.cuda.Stream()
    Fd = torch.tensor(stretch(3), device="cuda")
    with torch.cuda.stream(s):
        eager = [t.clone() for t in (*b.solve(Fd), *b.tangent(like=Fd))]
    s.synchronize()
    assert (eager[1] == 0).all() and (eager[3] == 0).all()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        out = (*b.solve(Fd), *b.tangent(like=Fd))
    for rep in range(3):
        with torch.cuda.stream(s):
            b.solve(Fd * 1.01)
            b.tangent(like=Fd)
        s.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for x, y in zip(out, eager):
            assert torch.equal(x, y), rep
    b.close()


def test_two_batches_at_once(rb, net1000):
    """64 RVEs of three parts on each of two streams, together more workgroups than CUs."""
    import torch
    o = dict(precision=rb.MIXED, mass=rb.MASS_SCALED, alpha=0.5, c=0.1, tol_abs=0.0, tol_rel=1e-12, n_max=200, check_every=8)
    batches = [rb.Batch(synth.pack([net1000] * 64), **o) for _ in range(2)]
    F = [torch.tensor(stretch(64, e), device="cuda") for e in (0.1, 0.12)]
    alone = []
    for b, f in zip(batches, F):
        alone.append(b.solve(f)[0].clone())
        torch.cuda.synchronize()
    out = [[], []]

    def work(i):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(5):
                out[i].append(batches[i].solve(F[i])[0])
        s.synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i in range(2):
        assert len(out[i]) == 5 and all(torch.equal(x, alone[i]) for x in out[i]), i
        batches[i].close()
