"""Calls whose natural grid would pass a limit of a launch (2^32 threads, 65535
blocks along y): they run, and give what small grids give."""
import numpy as np
import pytest
import torch

from paper_2412_09285_amd import fem
from paper_2412_09285_amd import workloads as W

pytestmark = pytest.mark.gpu


def pair():
    return fem.Problem.maxcut(2, [0], [1], [1.0])


def test_one_workgroup_per_replica_of_many():
    """17 instances of two nodes with 4,194,240 replicas: a workgroup of 64
    threads for each (instance, replica) would be 2^32 threads and more."""
    batch = fem.Problem.batch([pair() for _ in range(17)])
    R = 65535 * 64
    h0 = torch.randn(batch.n, R, device="cuda", generator=torch.Generator("cuda").manual_seed(1)) * 0.5
    out = []
    for problem, h in ((batch, h0), (pair(), h0[:2, :64].contiguous())):
        s = fem.Solver(problem, fem.default_params(replicas=h.shape[1], steps=10, energy_every=0))
        s.set_fields(h)
        s.step(3)
        out.append(s.fields(torch.empty_like(h)))
        s.sync()
        s.close()
    assert torch.equal(out[0][:2, :64], out[1])
    assert torch.isfinite(out[0]).all() and not torch.equal(out[0][32:], h0[32:])


def test_energies_of_many_instances_beside_a_large_one():
    """4,196,352 instances of two nodes and one of 140,000 (more than 128 tiles):
    a workgroup of 1024 threads per instance would be 2^32 threads and more."""
    many = fem.Problem.batch([pair()] * 2048)
    m = 140000
    path = fem.Problem.maxcut(m, np.arange(m - 1), np.arange(1, m), np.ones(m - 1, np.float32))
    batch = fem.Problem.batch([many] * 2049 + [path])
    h0 = torch.full((batch.n, 1), 0.25, device="cuda")
    out = []
    for problem, h in ((batch, h0), (pair(), h0[:2].contiguous()), (path, h0[:m].contiguous())):
        s = fem.Solver(problem, fem.default_params(replicas=1, steps=10))
        s.set_tile(1, 4, 4)
        s.set_fields(h)
        s.step(2)
        out.append(s.energies())
        s.close()
    for all_, one, last in zip(*out):
        # sums of two terms, and of some 10^5: float32 terms of one sign
        assert np.abs(all_[:-1] - one[0]).max() <= 4 * 2.0 ** -24 * np.abs(one[0]).max()
        assert np.abs(all_[-1] - last[0]).max() <= 8 * 2.0 ** -24 * np.abs(last[0]).max()


def test_training_on_millions_of_instances():
    """4,196,352 instances of one node: a workgroup of 1024 threads each would be
    2^32 threads and more.  Without neighbours the loss is a function of the
    logits alone, which the forward pass gives."""
    one = fem.Problem.maxcut(1, [], [])
    batch = fem.Problem.batch([fem.Problem.batch([one] * 2048)] * 2049)
    rng = np.random.default_rng(1)
    state = rng.standard_normal(batch.n).astype(np.float32)
    y = rng.integers(0, 2, batch.n).astype(np.int32)
    net = fem.MPNN(W.mpnn_init_weights(3))
    z = net.forward(batch, state, seed=5, draw=1).astype(np.float64)
    loss, g = net.train_step(batch, state, y, seed=5, draw0=1, lr=1e-3, want_grad=True)
    assert abs(loss - np.mean(np.logaddexp(0.0, z) - y * z)) <= 1e-5 * loss
    # d: the sum of dz over all nodes, float32 partial sums of some 2000 rows
    dz = (1.0 / (1.0 + np.exp(-z)) - y) / batch.n
    assert abs(g[-1] - dz.sum()) <= 2000 * 2.0 ** -24 * np.abs(dz).sum()


def test_column_blocks_of_the_chunk_sums():
    """1030 tiles, so that chunks are summed first, and 27000 replicas: more
    column blocks of energies and column sums than the launch has workgroups along y."""
    n, R, q = 1030, 27000, 2
    prob = fem.Problem.bmincut(n, np.arange(n - 1), np.arange(1, n), np.ones(n - 1, np.float32), q)
    h0 = torch.randn(n, R, q, device="cuda", generator=torch.Generator("cuda").manual_seed(2)) * 0.3
    out = []
    for r0, r1 in ((0, R), (R - 64, R)):
        h = h0[:, r0:r1].contiguous()
        s = fem.Solver(prob, fem.default_params(replicas=r1 - r0, steps=10, lam=0.01))
        s.set_tile(q, 1, 1)
        s.set_fields(h)
        s.step(3)
        out.append((s.fields(torch.empty_like(h)).cpu().numpy(), s.energies()))
        s.close()
    assert np.array_equal(out[0][0][:, -64:], out[1][0])
    for all_, some in zip(out[0][1], out[1][1]):
        assert np.allclose(all_[:, -64:], some, rtol=1e-12, atol=0)   # double sums of the same double terms
