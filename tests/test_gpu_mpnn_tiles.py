"""The network's training step at the edges of its tiles (sixteen nodes per
wave in the layer kernels, four rows per product and contiguous row ranges
per wave in the weight gradients), against the FP64 reference at the bar of
the other network tests."""
import numpy as np
import pytest

from oracle import mpnn as M
from paper_2412_09285_amd import fem
from paper_2412_09285_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(1,), (2, 1), (3, 5, 7), (15,), (17, 64), (65, 1, 62), (1000, 4001), (9, 33000)])
def test_train_step(sizes):
    graphs = [W.random_sparse_graph(n, min(3 * n, n * (n - 1) // 4), seed=n, weights="pm1") for n in sizes]
    off = np.cumsum([0] + [g.n for g in graphs]).astype(np.int64)
    u, v, w = (np.concatenate([getattr(g, k) + (o if k != "w" else 0) for g, o in zip(graphs, off)]) for k in "uvw")
    ops = M.GraphOps(int(off[-1]), u, v, w)
    batch = fem.Problem.batch([fem.Problem.maxcut(g.n, g.u, g.v, g.w) for g in graphs])
    rng = np.random.default_rng(len(sizes))
    st = (rng.standard_normal(batch.n) * 2).astype(np.float32)
    y = rng.integers(0, 2, size=batch.n).astype(np.int32)
    theta = W.mpnn_init_weights(3)
    net = fem.MPNN(theta)
    loss, g = net.train_step(batch, st, y, seed=5, draw0=1, lr=1e-3, want_grad=True)
    Lr, gr, _ = M.batch_loss_and_grad(ops, off, st, y, theta, 5, 1)
    assert loss == pytest.approx(Lr, rel=1e-5)
    assert np.linalg.norm(g - gr) <= 1e-5 * np.linalg.norm(gr)
    assert np.abs(g - gr).max() <= 1e-5 * np.abs(gr).max()
    # a repeated first step from the same parameters is the same step
    th = net.params()
    net.set_params(theta)
    assert net.train_step(batch, st, y, seed=5, draw0=1, lr=1e-3) == loss
    assert np.array_equal(net.params(), th)
