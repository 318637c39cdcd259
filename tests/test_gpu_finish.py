"""The reductions behind a step (energies, bMinCut column sums) in one launch
and over chunks of tiles: launch shapes on both sides of the tile limit give
the same fields bit for bit and the same energies, for every number of
states and for replica counts around the columns of a workgroup."""
import numpy as np
import pytest

from paper_2412_09285_amd import fem
from paper_2412_09285_amd import workloads as W

pytestmark = pytest.mark.gpu

N = 16500   # a one-wave tile of up to sixteen rows: more than 1024 tiles


def run(prob, R, q, tile, **kw):
    h0 = W.initial_fields(prob.n, R, seed=2, q=q, std=0.3)
    s = fem.Solver(prob, fem.default_params(replicas=R, steps=20, energy_every=1, **kw))
    s.set_tile(*tile)
    s.set_fields(h0)
    s.step(3)
    return s.fields(), s.energies()


@pytest.mark.parametrize("q,R", [(2, 3), (2, 9), (4, 33), (8, 16), (16, 5), (32, 2)])
def test_bmincut(q, R):
    g = W.rgg_3d(N, 6.0, seed=1)
    prob = fem.Problem.bmincut(g.n, g.u, g.v, g.w, q)
    many, few = (run(prob, R, q, t, lam=0.01) for t in ((q, 1, 1, 0, 0), (q, 2, 64, 0, 0)))
    assert np.array_equal(many[0], few[0])
    for a, b in zip(many[1], few[1]):      # double sums of the same double terms
        assert np.allclose(a, b, rtol=1e-12, atol=0)


@pytest.mark.parametrize("kind", ["maxcut", "maxsat"])
@pytest.mark.parametrize("R", [1, 7, 8, 70])
def test_one_logit(kind, R):
    if kind == "maxcut":
        g = W.random_sparse_graph(N, 2 * N, seed=4, weights="pm1")
        prob, scale = fem.Problem.maxcut(g.n, g.u, g.v, g.w), 2.0 * N
    else:
        cnf = W.random_ksat(N, 3 * N, 3, seed=4)
        prob, scale = fem.Problem.from_cnf(cnf), 3.0 * N
    many, few = (run(prob, R, 1, t) for t in ((1, 1, 1, 0, 4), (1, 4, 64, 0, 0)))
    assert np.array_equal(many[0], few[0])
    # float32 sums over the (at most 64) rows of a lane
    for a, b, m in zip(many[1][:2], few[1][:2], (scale, N)):
        assert np.all(np.abs(a - b) <= 64 * 2.0 ** -24 * m)
