"""Resident anneals (small one-logit instances that stay on one compute unit)
against the row-tiled kernels, which an explicit launch shape selects: fields,
gradients and anytime bests bit for bit, energies up to the rounding of their
float32 per-lane terms; ranges split anywhere; batches in which some
instances are resident and others are not."""
# (A batch is resident as a whole or row-tiled as a whole: test_mixed_batch holds
# batches that are row-tiled against their instances alone, some of which are
# resident; test_gpu_resident_ranges.py has batches that are resident.)
import numpy as np
import pytest
import torch

from paper_2412_09285_amd import fem
from paper_2412_09285_amd import workloads as W

pytestmark = pytest.mark.gpu

TILE = (1, 4, 4, 0, 0)   # one value per lane fits every replica count


def graph(n, edges, weights, seed=1):
    edges = min(edges, n * (n - 1) // 2)
    g = W.er_graph_m(n, edges, seed=seed, weights="one" if weights == "real" else weights)
    w = W.rng_for(seed + 1).standard_normal(edges).astype(np.float32) if weights == "real" else g.w
    return fem.Problem.maxcut(n, g.u, g.v, w), float(np.abs(w.astype(np.float64)).sum())


def formula(n, m, kmax, seed=1):
    """Clauses of 1..kmax distinct variables (as many as n allows)."""
    rng = W.rng_for(seed)
    lits, off = [], [0]
    for _ in range(m):
        k = min(int(rng.integers(1, kmax + 1)), n)
        v = rng.choice(n, size=k, replace=False) + 1
        lits.extend((v * np.where(rng.integers(0, 2, k) == 1, 1, -1)).tolist())
        off.append(len(lits))
    return fem.Problem.maxsat(n, np.array(off), np.array(lits, np.int32)), float(m)


def compare(prob, u_scale, R, splits, seed=3, std=0.5, **kw):
    h0 = W.initial_fields(prob.n, R, seed=seed, std=std)
    out = []
    for tiled in (False, True):
        s = fem.Solver(prob, fem.default_params(replicas=R, steps=40, keep_grad=1, **kw), stream=torch.cuda.Stream())
        if tiled:
            s.set_tile(*TILE)
        s.set_fields(h0)
        for n in splits:
            if n % 2:
                s.step(n)
            else:
                s.run_until(s.t + n)
        r = dict(h=s.fields(), g=s.last_grad(), state=s.get_state(), sig=s.round(), best=s.best())
        if kw.get("energy_every", 1):
            r["e"] = s.energies()
        if kw.get("eval_every"):
            r["any"] = s.anytime_best()
        s.close()
        out.append(r)
    a, b = out
    assert np.array_equal(a["h"], b["h"]) and np.array_equal(a["g"], b["g"])
    assert np.array_equal(a["sig"], b["sig"]) and a["state"] == b["state"]
    assert all(np.array_equal(x, y) for x, y in zip(a["best"], b["best"]))
    if "any" in a:
        assert np.array_equal(a["any"], b["any"])
    if "e" in a:
        # at most eight float32 additions per term on either side, each term
        # also rounded once: 20 units of 2^-24 of the summed magnitudes
        tol = 20 * 2.0 ** -24
        for b_ in range(prob.n_inst):
            assert np.all(np.abs(a["e"][0][b_] - b["e"][0][b_]) <= tol * (2 * u_scale + 1))
            assert np.all(np.abs(a["e"][1][b_] - b["e"][1][b_]) <= tol * prob.n)


@pytest.mark.parametrize("n,edges,R,weights,dtype", [
    (1, 0, 1, "one", "f32"), (2, 1, 7, "pm1", "bf16"), (63, 300, 9, "real", "f32"), (64, 64, 8, "pm1", "f32"),
    (65, 2000, 16, "one", "bf16"), (200, 900, 33, "real", "bf16"), (513, 8000, 5, "pm1", "f32"),
    (1024, 5000, 12, "pm1", "f32"), (1025, 20000, 3, "one", "f32"), (2049, 30000, 4, "real", "f32"),
    (4097, 12300, 3, "pm1", "bf16"), (700, 60000, 5, "pm1", "f32"), (2100, 90000, 3, "real", "bf16"), (8190, 20000, 2, "pm1", "f32"), (8191, 20000, 2, "pm1", "f32")])
def test_maxcut(n, edges, R, weights, dtype):
    prob, scale = graph(n, edges, weights)
    compare(prob, scale, R, (1, 6, 3), marginal_dtype=fem.BF16 if dtype == "bf16" else fem.F32, eval_every=4,
            energy_every=3)


@pytest.mark.parametrize("n,edges,R,weights", [(1, 0, 3, "one"), (130, 600, 40, "pm1"), (1500, 20000, 33, "one"),
                                               (3000, 9000, 10, "real"), (8190, 12000, 2, "pm1"),
                                               (900, 100000, 3, "one")])
@pytest.mark.parametrize("opt", [fem.OPT_RMSPROP, fem.OPT_SGD])
def test_manipulated(n, edges, R, weights, opt):
    prob, scale = graph(n, edges, weights)
    compare(prob, scale, R, (2, 5), gradient=fem.GRAD_MANIPULATED, energy_every=0, gamma_grad=1.5, optimizer=opt,
            lr=0.05, momentum=0.5, eval_every=5)


@pytest.mark.parametrize("n,m,kmax,R,dtype", [(1, 3, 1, 5, "f32"), (3, 10, 4, 16, "f32"), (64, 500, 3, 9, "bf16"),
                                              (200, 1200, 3, 64, "f32"), (300, 900, 4, 17, "bf16"),
                                              (1100, 9000, 3, 6, "f32"), (2500, 8000, 4, 3, "f32"),
                                              (4088, 9000, 2, 2, "f32"), (4089, 9000, 2, 2, "f32"),
                                              (1100, 30000, 3, 4, "f32"), (2100, 25000, 4, 3, "f32")])
def test_maxsat(n, m, kmax, R, dtype):
    prob, scale = formula(n, m, kmax)
    compare(prob, scale, R, (4, 1, 3), marginal_dtype=fem.BF16 if dtype == "bf16" else fem.F32, eval_every=3,
            energy_every=2)


@pytest.mark.parametrize("n,edges,R,eval_every", [(4097, 9000, 3, 0), (8190, 12000, 2, 0), (5000, 20000, 2, 16),
                                                  (5000, 20000, 2, 15)])
def test_eight_rows_per_thread(n, edges, R, eval_every):
    """Resident without read-outs or 16 steps apart, row-tiled below."""
    prob, scale = graph(n, edges, "pm1")
    compare(prob, scale, R, (1, 16, 4), eval_every=eval_every)


@pytest.mark.parametrize("kind", ["maxcut", "manip", "maxsat"])
def test_mixed_batch(kind):
    """Instances on both sides of the size rule: an instance alone (resident,
    if it is small) and inside the batch (row-tiled) gives the same fields to
    the bit; energies meet within the float32 terms that they are sums of."""
    kw = dict(eval_every=4, energy_every=2)
    if kind == "maxsat":
        made = [formula(n, 4 * n, 3, seed=n) for n in (90, 9000, 1500, 300)]
    else:
        made = [graph(n, 4 * n, "pm1", seed=n) for n in (90, 9000, 1500, 300, 4000)]
        if kind == "manip":
            kw = dict(kw, gradient=fem.GRAD_MANIPULATED, energy_every=0)
    parts = [p for p, _ in made]
    batch = fem.Problem.batch(parts)
    R = 20
    compare(batch, max(s for _, s in made), R, (5, 4), **kw)
    h0 = W.initial_fields(batch.n, R, seed=5)
    off = batch.instance_offsets()
    both = []
    for prob, h in [(batch, h0)] + [(p, h0[i:j].copy()) for p, i, j in zip(parts, off[:-1], off[1:])]:
        s = fem.Solver(prob, fem.default_params(replicas=R, steps=40, **kw), stream=torch.cuda.Stream())
        s.set_fields(h)
        s.run_until(9)
        both.append((s.fields(), s.anytime_best(), s.energies() if kind != "manip" else ()))
        # the captured range again, with eager steps and getters in between
        for _ in range(3):
            s.set_fields(h)
            s.run_until(9)
            assert np.array_equal(s.fields(), both[-1][0]) and np.array_equal(s.anytime_best(), both[-1][1])
            s.step(1)
    hb, bb, eb = both[0]
    for k, (h, b, e) in enumerate(both[1:]):
        assert np.array_equal(h, hb[off[k]:off[k + 1]]) and np.array_equal(b[0], bb[k])
        # 20 units of 2^-24 as in compare; F = U - S / beta with beta >= 0.01
        tol = 20 * 2.0 ** -24 * np.array([2 * made[k][1] + 1, h.shape[0], 2 * made[k][1] + 1 + 100 * h.shape[0]])
        for x, y, bound in zip(e, eb, tol):
            assert np.abs(x[0] - y[k]).max() <= bound


def test_tuning_of_a_mixed_batch(tmp_path, monkeypatch):
    """The tuner times shapes for a batch with one instance too large to be
    resident, and restores the state."""
    monkeypatch.setenv("FEM_TUNE_CACHE", str(tmp_path / "tune.txt"))
    batch = fem.Problem.batch([graph(n, 3 * n, "pm1", seed=n)[0] for n in (9000, 500)])
    h0 = W.initial_fields(batch.n, 16, seed=1)
    out = []
    for tune in (False, True):
        s = fem.Solver(batch, fem.default_params(replicas=16, steps=40), stream=torch.cuda.Stream())
        s.set_fields(h0)
        s.step(3)
        if tune:
            tile = s.tune(trial_steps=1, use_cache=False)
            assert tile == s.tile() == s.tune(trial_steps=1, use_cache=True)
        s.run_until(9)
        out.append(s.fields())
    assert np.array_equal(*out)
