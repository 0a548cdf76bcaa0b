"""Paths of the relaxation and the tangent over several workgroups per RVE that a single
ordinary call does not take: teams that give up in a warm start."""
import pytest

from gpu_common import require_gpu
from paper_2306_09427_amd import synth
from test_gpu_spread import same, stretch

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
