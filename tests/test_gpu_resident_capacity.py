"""RVEs that fill every fiber slot of a register-resident build run on that build."""
import pytest

from gpu_common import require_gpu
from paper_2306_09427_amd import binding as rb, synth
from test_gpu_resident_edges import check, pieces


@pytest.mark.parametrize("precision", [0, 1])
def test_indices_of_full_builds(precision):
    """The zero force slot behind the last fiber lies inside the LDS arrays."""
    for n_fib in (1024, 2048, 3072, 3967, 4095, 4096, 6144):
        rb.check_indexing(synth.pack([pieces(n_fib), pieces(n_fib, hubs=[5, 9], seed=1)]), precision)


# (precision, threads_per_rve, fibers): the largest RVE of the thread count
@pytest.mark.gpu
@pytest.mark.parametrize("precision,threads,n_fib", [(1, 256, 1024), (1, 512, 3072), (1, 768, 3072), (1, 1024, 6144),
                                                     (1, 0, 6144), (0, 256, 1024)])
def test_full_builds(precision, threads, n_fib):
    nets = [pieces(n_fib), pieces(n_fib, hubs=[5, 9], seed=1)]
    d = check(require_gpu(), nets, precision, threads_per_rve=threads)
    assert d.startswith("resident(") and ":2" in d and "streamed" not in d, d
