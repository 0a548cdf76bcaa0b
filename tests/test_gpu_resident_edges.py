"""Register-resident kernels at the edges of their slots and tables.

Networks made of independent pieces with a known fiber count: bent two-fiber
chains (one free node each) and hubs (one free node of a given degree), so a
network ends exactly at, before or after a build's last fiber slot or a wave's
last lane, and holds nodes whose incidences fill, or pass, the on-chip table of
degrees above 4 and boundary lists longer than the boundary table.  Every
stress is compared with the oracle's.
"""
import numpy as np
import pytest

from gpu_common import rel_err, require_gpu
from paper_2306_09427_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rb():
    return require_gpu()


def pieces(n_fib, hubs=(), seed=0, shared=0):
    """A network of exactly n_fib fibers: hubs of the given degrees, then bent
    two-fiber chains, then single fibers between boundary nodes.  shared: that
    many chains start at one common boundary node."""
    rng = np.random.default_rng([n_fib, seed])
    X, bnd, fib = [], [], []

    def node(p, b):
        X.append(p)
        bnd.append(b)
        return len(X) - 1

    def face():
        p = rng.random(3)
        k = rng.integers(3)
        p[k] = rng.integers(2)
        return p

    left = n_fib
    for d in hubs:
        c = node(0.3 + 0.4 * rng.random(3), 0)
        for _ in range(d):
            fib.append((c, node(face(), 1)))
        left -= d
    common = node(np.array([0.0, 0.5, 0.5]), 1) if shared else None
    while left >= 2:
        a = common if shared > 0 else node(np.array([0.0, *rng.random(2)]), 1)
        shared -= 1
        b = node(np.array([1.0, *rng.random(2)]), 1)
        m = node(0.5 * (X[a] + X[b]) + 0.05 * rng.standard_normal(3), 0)
        fib += [(a, m), (m, b)]
        left -= 2
    if left:
        fib.append((node(np.array([0.0, *rng.random(2)]), 1), node(np.array([1.0, *rng.random(2)]), 1)))
    assert len(fib) == n_fib
    return synth.Network(np.array(X), np.array(bnd, np.uint8), np.array(fib, np.int32))


def check(rb, nets, precision, **kw):
    import oracle
    batch = synth.pack(nets)
    rng = np.random.default_rng(len(nets))
    F = np.diag([1.15, 1.05, 1.05]) + 0.02 * rng.standard_normal((len(nets), 3, 3))
    fp64 = precision == rb.FP64
    opts = dict(tol_rel=1e-9 if fp64 else 1e-5, n_max=20000)
    b = rb.Batch(batch, precision=precision, law=rb.LAW_EXP, mass=rb.MASS_SCALED, alpha=0.5, c=0.5, tol_abs=0.0,
                 check_every=4, **opts, **kw)
    sig, st = b.solve(F)
    sig2, st2 = b.solve(F)
    d = b.describe()
    b.close()
    ref = oracle.solve_batch(batch, F, 0.5, oracle.make_opts(law=oracle.EXP, mass=1, alpha=0.5, tol_abs=0.0, **opts))
    assert np.array_equal(sig, sig2) and np.array_equal(st, st2), "a second solve differs"
    assert (st == 0).all() and (ref["status"] == 0).all(), (st, ref["status"])
    err = rel_err(sig, ref["sigma"])
    assert np.all(err < (1e-5 if fp64 else 1e-4)), (d, err.max(), int(err.argmax()))
    return d


COUNTS = [1, 2, 63, 64, 65, 127, 511, 512, 513, 1022, 1023, 1024, 1025, 2046, 2047, 2048, 2049, 3070, 3071, 3072, 3073,
          3966, 3967, 3968, 3969, 4094, 4095, 4096]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("many", [False, True])
def test_fiber_counts_at_slot_edges(rb, precision, many):
    """many: with more RVEs than CUs the builds are chosen for throughput."""
    nets = [pieces(n) for n in COUNTS]
    small = [pieces(65, seed=k) for k in range(300 if many else 0)]
    d = check(rb, nets + small, precision)
    assert "resident" in d


@pytest.mark.parametrize("precision", [0, 1])
def test_degrees_and_boundary_lists(rb, precision):
    nets = [pieces(40, hubs=[5]), pieces(60, hubs=[4, 5, 6, 7, 8]), pieces(200, hubs=[8, 9, 12, 13, 16, 17, 30]),
            pieces(1000, hubs=[5] * 100 + [9] * 3), pieces(900, hubs=[40] * 20),          # tables full or past their end
            pieces(300, shared=3), pieces(1023, hubs=[6] * 64, shared=100), pieces(2047, hubs=[5, 300])]
    for threads in (0, 512, 1024):
        check(rb, nets, precision, threads_per_rve=threads)


def test_six_slot_builds(rb):
    d = check(rb, [pieces(n) for n in (4097, 6142, 6143)], rb.MIXED)
    assert "resident(1024,6,3):3" in d


@pytest.mark.parametrize("precision", [0, 1])
def test_kinetic_builds_at_slot_edges(rb, precision):
    """Kinetic builds: the same equilibria (these networks have one each)."""
    nets = [pieces(n, hubs=[5, 9]) for n in (64, 1023, 1024, 2047, 3071, 3967, 4095)]
    batch = synth.pack(nets)
    F = np.broadcast_to(np.diag([1.15, 1.05, 1.05]), (len(nets), 3, 3)).copy()
    out = []
    for damping in (0, 1):
        b = rb.Batch(batch, precision=precision, law=rb.LAW_EXP, mass=rb.MASS_SCALED, alpha=0.5, c=0.5, tol_abs=0.0,
                     tol_rel=1e-9 if precision == rb.FP64 else 1e-5, n_max=20000, damping=damping)
        sig, st = b.solve(F)
        b.close()
        assert (st == 0).all(), st
        out.append(sig)
    assert np.all(rel_err(out[1], out[0]) < (1e-5 if precision == rb.FP64 else 1e-4))
