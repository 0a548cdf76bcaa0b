"""A caller-owned workspace on a batch whose tangent runs over several workgroups per RVE.

The size is asked for, and the workspace bound, before the first tangent: it has to
hold what the first tangent and VJP need, and stay the reported size after them.
"""
import numpy as np
import pytest

from gpu_common import require_gpu
from paper_2306_09427_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("small", [0, 3])
def test_size_bound_before_the_first_tangent_is_enough(small):
    rb = require_gpu()
    import torch
    nets = [synth.voronoi_network(1000, [41, 0, 0])] + [synth.voronoi_network(60, [41, 5, k]) for k in range(small)]
    assert nets[0].n_free > 4096
    F = np.broadcast_to(np.diag([1.1, 0.97, 0.97]), (len(nets), 3, 3)).copy()
    g = np.random.default_rng(5).standard_normal(F.shape)
    o = dict(precision=rb.MIXED, mass=rb.MASS_SCALED, alpha=0.5, c=0.1, tol_abs=0.0, tol_rel=1e-5, n_max=20000,
             check_every=8)

    def run(bind):
        b = rb.Batch(synth.pack(nets), **o)
        if bind:
            need = b.workspace_size()
            buf = torch.empty(need + 256, dtype=torch.uint8, device="cuda")
            off = -buf.data_ptr() % 256
            b.bind_workspace(buf[off:off + need])
        sig, st = b.solve(F)
        out = [sig, st, *b.tangent(), *b.vjp(g)]
        if bind:
            assert b.workspace_size() == need
            b.bind_workspace(None)
            b.bind_workspace(buf[off:off + need])   # the same buffer again
            out += [*b.tangent(), *b.vjp(g)]
        b.close()
        return out

    own, bound = run(False), run(True)
    assert (own[1] == 0).all() and (own[3] == 0).all() and (own[5] == 0).all()
    for x, y in zip(own + own[2:], bound):
        assert np.array_equal(x, y)
