"""Read-out on bit words and the best replica chosen on the device, against the
byte evaluation (fem_eval_int) of the rounded fields and the scores by
definition: replica counts around the word and segment sizes, rows longer
than a counter holds, every clause length, batches, and bMinCut's scores."""
import numpy as np
import pytest
import torch

from paper_2412_09285_amd import fem
from paper_2412_09285_amd import workloads as W

pytestmark = pytest.mark.gpu


def check(prob, R, seed=1, lam=0.3):
    rng = W.rng_for(seed)
    q = prob.q if prob.kind == fem.BMINCUT else 1
    h = rng.standard_normal((prob.n, R) if q == 1 else (prob.n, R, q)).astype(np.float32)
    h[rng.random(h.shape) < 0.1] = 0.0                  # ties
    s = fem.Solver(prob, fem.default_params(replicas=R, steps=4, eval_every=2, energy_every=0, lam=lam),
                   stream=torch.cuda.Stream())
    for _ in range(2):
        s.set_fields(h)
        rep, val, sig = s.best()
        sigma = s.round()
        v, sizes = prob.eval_int(sigma)
        off = prob.instance_offsets()
        for b in range(prob.n_inst):
            score = -v[b] if prob.kind == fem.MAXCUT else v[b].astype(np.float64)
            if prob.kind == fem.BMINCUT:
                score = 2.0 * v[b] + lam * (np.sum(sizes[b].astype(np.float64) ** 2, axis=1) - (off[b + 1] - off[b]))
            assert rep[b] == int(np.argmin(score)) and val[b] == v[b][rep[b]]
            assert np.array_equal(sig[off[b]:off[b + 1]], sigma[rep[b], off[b]:off[b + 1]])
        # the anytime best is the evaluation of the fields it was taken at
        s.run_until(2)
        v, sizes = prob.eval_int(s.round())
        if prob.kind != fem.BMINCUT:
            assert np.array_equal(s.anytime_best(), v)


@pytest.mark.parametrize("n,edges,R", [(1, 0, 1), (2, 1, 31), (300, 900, 32), (301, 40000, 33), (700, 200000, 100),
                                       (9000, 20000, 64), (9000, 40000, 257), (50, 300, 2100)])
def test_cut(n, edges, R):
    g = W.er_graph_m(n, min(edges, n * (n - 1) // 2), seed=n, weights="pm1")
    check(fem.Problem.maxcut(g.n, g.u, g.v, g.w), R)


@pytest.mark.parametrize("n,m,kmax,R", [(1, 2, 1, 3), (40, 400, 3, 32), (500, 20000, 3, 65), (600, 3000, 4, 40),
                                        (9000, 30000, 4, 16), (30, 200, 4, 2100)])
def test_unsatisfied(n, m, kmax, R):
    rng = W.rng_for(n)
    lits, off = [], [0]
    for _ in range(m):
        v = rng.choice(n, size=min(int(rng.integers(1, kmax + 1)), n), replace=False) + 1
        lits.extend((v * np.where(rng.integers(0, 2, v.size) == 1, 1, -1)).tolist())
        off.append(len(lits))
    check(fem.Problem.maxsat(n, np.array(off), np.array(lits, np.int32)), R)


@pytest.mark.parametrize("R", [5, 32, 70])
def test_batch(R):
    parts = []
    for k, n in enumerate((60, 9100, 1, 2500)):
        g = W.er_graph_m(n, min(3 * n, n * (n - 1) // 2), seed=k, weights="pm1")
        parts.append(fem.Problem.maxcut(g.n, g.u, g.v, g.w))
    check(fem.Problem.batch(parts), R)


@pytest.mark.parametrize("q,R", [(2, 7), (8, 33)])
def test_bmincut_and_real_weights(q, R):
    g = W.rgg_3d(900, 8.0, seed=q)
    check(fem.Problem.bmincut(g.n, g.u, g.v, g.w, q), R)
    w = np.round(W.rng_for(3).standard_normal(g.u.size) * 5).astype(np.float32)   # integral, not +-1
    check(fem.Problem.maxcut(g.n, g.u, g.v, w), R)


@pytest.mark.parametrize("n,edges,R", [(129, 129 * 64, 1), (129, 128 * 64, 32), (700, 700 * 699 // 2, 33), (1500, 300000, 64),
                                       (2100, 2100 * 2099 // 2, 1), (2100, 2100 * 2099 // 2, 100), (2100, 2000000, 257)])
def test_rows_shared_by_several_lanes(n, edges, R):
    """Mean degrees around 64 and far above, where the lanes of a row split its entries."""
    g = W.er_graph_m(n, edges, seed=n, weights="pm1")
    check(fem.Problem.maxcut(g.n, g.u, g.v, g.w), R)


@pytest.mark.parametrize("k", [3, 4])
def test_clauses_shared_by_several_lanes(k):
    check(fem.Problem.from_cnf(W.random_ksat(60, 9000, k, seed=k)), 40)
