"""Block shapes of the dense-W step on the GPU: ragged blocks of every kernel
against the FP64 oracle, and the kernels of the two block sizes of each weight
type against one another.

The int8 products are exact and the FP64 products sum each quarter of the
contraction in the same order in both block sizes, so a replica's fields don't
depend on how many others run beside it: those comparisons are bit for bit.
Gradients and fields meet the oracle within the 1e-5 of the other dense tests.
"""
import numpy as np
import pytest

from paper_2412_09285_amd import fem
from paper_2412_09285_amd import workloads as W
from test_gpu_dense import K2000_OPT, lockstep_dense

pytestmark = pytest.mark.gpu


def _graph(n, real, seed):
    g = W.complete_pm1(n, seed=seed)
    if real:
        g.w = (g.w * np.random.default_rng(seed).uniform(0.5, 1.5, size=g.n_edges)).astype(np.float32)
    return g


@pytest.mark.parametrize("real", [False, True])
@pytest.mark.parametrize("n,R", [(15, 17), (16, 16), (31, 33), (33, 31), (127, 65), (129, 64), (385, 1)])
def test_ragged_blocks(n, R, real):
    lockstep_dense(_graph(n, real, seed=n), R=R, T=100, n_steps=8, seed=n + R, tag=f"dense blocks n{n} R{R} real{real}")


@pytest.mark.parametrize("real,n,R", [(False, 250, 6150), (True, 250, 645), (True, 140, 1030)])
def test_block_sizes_agree(real, n, R):
    """R replicas run in the larger blocks, their first and last 40 alone in the smaller ones."""
    prob = fem.Problem.maxcut_dense(W.dense_matrix(_graph(n, real, seed=n)))
    h0 = W.initial_fields(n, R, seed=R)

    def run(cols):
        s = fem.Solver(prob, fem.default_params(replicas=cols.size, steps=1000, energy_every=1, **K2000_OPT))
        s.set_fields(np.ascontiguousarray(h0[:, cols]))
        s.run_until(6)
        return s.fields(), np.array(s.energies())

    allr = np.arange(R)
    f, e = run(allr)
    for cols in (allr[:40], allr[-40:]):
        fs, es = run(cols)
        assert np.array_equal(f[:, cols], fs)
        # sums of the same float64 terms over blocks of other sizes: at most a
        # few hundred roundings of 2^-53 of the sum of magnitudes (n^2 + n)
        assert np.abs(e[..., cols] - es).max() <= 1e-13 * (n * n + n) * 10
