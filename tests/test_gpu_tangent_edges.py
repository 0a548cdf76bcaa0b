"""On-chip tangent and VJP kernels at the edges of their slots and tables,
against the streamed kernel (one wavefront per right-hand side)."""
import numpy as np
import pytest

from gpu_common import require_gpu
from paper_2306_09427_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rb():
    return require_gpu()


def lattice(n, drop, seed):
    """A perturbed cubic lattice without its last `drop` free nodes' fibers:
    (n - 1)^3 - drop free nodes, all of degree up to 6 (every record table full)."""
    net = synth.lattice_network(n)
    rng = np.random.default_rng(seed)
    X = net.X + np.where(net.is_bnd[:, None], 0.0, 0.1 / n) * rng.standard_normal(net.X.shape)
    free = np.nonzero(net.is_bnd == 0)[0]
    gone = free[len(free) - drop:]
    keep = ~np.isin(net.fib, gone).any(axis=1)
    fib = net.fib[keep]
    used = np.zeros(len(X), bool)
    used[fib.ravel()] = True
    new = np.cumsum(used) - 1
    return synth.Network(X[used], net.is_bnd[used], new[fib].astype(np.int32))


NETS = {
    "lattice512": lambda: lattice(9, 0, 1), "lattice511": lambda: lattice(9, 1, 2), "lattice1000": lambda: lattice(11, 0, 3),
    "lattice1728": lambda: lattice(13, 0, 4), "lattice8": lambda: lattice(3, 0, 5),
    "voronoi60": lambda: synth.voronoi_network(60, [31, 0, 0]), "voronoi250": lambda: synth.voronoi_network(250, [31, 1, 0]),
    "voronoi400": lambda: synth.voronoi_network(400, [31, 2, 0]),
}


@pytest.mark.parametrize("copies", [1, 40])
def test_on_chip_tangent_and_vjp(rb, copies):
    """copies 1: workgroups on CUs of their own; 40: several per CU, and more tasks than workgroups."""
    nets = [f() for f in NETS.values()] * copies
    F = np.broadcast_to(np.diag([1.1, 1.08, 1.06]), (len(nets), 3, 3)).copy()
    F[:, 0, 1] = 0.01 * np.arange(len(nets)) / len(nets)
    g = np.random.default_rng(0).standard_normal((len(nets), 3, 3))
    opts = dict(c=0.3, precision=rb.FP64, law=rb.LAW_EXP, mass=rb.MASS_SCALED, alpha=0.5, tol_abs=0.0, tol_rel=1e-9,
                n_max=40000, check_every=8, cg_tol=1e-9)
    out = []
    for engine in (rb.ENGINE_AUTO, rb.ENGINE_STREAMED):
        b = rb.Batch(synth.pack(nets), **opts)
        if not out:
            _, st = b.solve(F)
            assert (st == 0).all(), st
            state = b.export_state()
        b.set_opts(engine=engine, **opts)
        b.import_state(*state)   # the same state for both
        C, cs = b.tangent()
        C2, _ = b.tangent()
        gF, gs = b.vjp(g)
        assert np.array_equal(C, C2)
        assert (cs == 0).all() and (gs == 0).all(), (cs, gs)
        b.close()
        out.append((C, gF))
    scale = np.abs(out[1][0]).max(axis=(1, 2))
    assert np.all(np.abs(out[0][0] - out[1][0]).max(axis=(1, 2)) < 1e-7 * scale)
    want = np.einsum("rp,rpq->rq", g.reshape(-1, 9), out[0][0]).reshape(-1, 3, 3)
    assert np.all(np.abs(out[0][1] - want).max(axis=(1, 2)) < 1e-6 * scale * np.abs(g).max())
