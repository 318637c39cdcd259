"""Solvers of small instances whose step ranges change length: long ones run on
one compute unit per replica, short ones on the row-tiled kernels, and the two
alternate on the same state; batches of several workgroup sizes, which run on
side streams; ranges inside a caller's graph.  Everything is compared with a
solver that an explicit launch shape keeps on the row-tiled kernels: fields,
moments, read-outs and anytime bests bit for bit."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest
import torch

from paper_2412_09285_amd import fem
from paper_2412_09285_amd import workloads as W

pytestmark = pytest.mark.gpu

TILE = (1, 4, 2, 0, 0)


def graph(n, deg, weights="pm1", seed=1):
    m = min(n * deg // 2, n * (n - 1) // 2)
    g = W.er_graph_m(n, m, seed=seed, weights="one" if weights == "real" else weights)
    w = W.rng_for(seed + 1).standard_normal(m).astype(np.float32) if weights == "real" else g.w
    return fem.Problem.maxcut(n, g.u, g.v, w)


def formula(n, m, k=3, seed=1):
    return fem.Problem.from_cnf(W.random_ksat(n, m, k, seed=seed))


def problem(kind):
    if kind == "batch":
        return fem.Problem.batch([graph(n, 6, seed=n) for n in (90, 300, 700, 1500, 3000)])
    if kind == "sat batch":
        return fem.Problem.batch([formula(n, 4 * n, seed=n) for n in (90, 300, 700, 1500, 3000)])
    return {"rows 1": lambda: graph(900, 20), "rows 2": lambda: graph(2000, 20), "rows 4": lambda: graph(3500, 8, "real"),
            "rows 8": lambda: graph(5000, 4), "sat": lambda: formula(1500, 6300),
            "manip": lambda: graph(2000, 20, "one"), "manip batch": lambda: problem("batch"),
            "real": lambda: graph(300, 12, "real")}[kind]()


def solver(prob, R, kind, tiled, **kw):
    if kind.startswith("manip"):
        kw.update(gradient=fem.GRAD_MANIPULATED, energy_every=0)
    s = fem.Solver(prob, fem.default_params(replicas=R, steps=400, keep_grad=1, **kw), stream=torch.cuda.Stream())
    if tiled:
        s.set_tile(*TILE)
    return s


@pytest.mark.parametrize("kind", ["rows 1", "rows 2", "rows 4", "rows 8", "sat", "manip", "real", "batch", "manip batch",
                                  "sat batch"])
@pytest.mark.parametrize("eval_every,dtype", [(0, fem.F32), (3, fem.BF16), (20, fem.F32)])
def test_ranges_of_changing_length(kind, eval_every, dtype):
    prob = problem(kind)
    R = 11
    h0 = W.initial_fields(prob.n, R, seed=3, std=0.4)
    h1 = W.initial_fields(prob.n, R, seed=4, std=0.4)
    a, b = (solver(prob, R, kind, tiled, eval_every=eval_every, marginal_dtype=dtype) for tiled in (False, True))
    for s in (a, b):
        s.set_fields(torch.from_numpy(h0).cuda())
    blob = None
    plan = [1, 1, 40, 2, 33, 3, 1, "graph", 50, "graph", "save", 1, 35, "load", 1, "set", 1, 2, 40, "graph", 5, 17, 34,
            "load", 36]
    for op in plan:
        for s in (a, b):
            if op == "graph":          # short ranges twice, the second time from a replayed graph
                t = s.t
                st = s.get_state()
                s.capture(t + 2)
                s.run_until(t + 2)
                s.step(35)
                s.set_state(st)
                s.run_until(t + 2)
            elif op == "save":
                blob = b.get_state()
            elif op == "load":
                s.set_state(blob)
            elif op == "set":
                s.set_fields(h1)
            else:
                s.step(op)
        assert a.t == b.t and a.get_state() == b.get_state(), op
        if op not in ("save", "load", "set"):
            assert np.array_equal(a.last_grad(), b.last_grad()), op
        if eval_every:
            assert np.array_equal(a.anytime_best(), b.anytime_best()), op
    assert np.array_equal(a.round(), b.round())
    assert all(np.array_equal(x, y) for x, y in zip(a.best(), b.best()))


@pytest.mark.parametrize("kind", ["rows 2", "rows 4", "rows 8", "sat", "batch"])
def test_short_ranges_take_the_row_tiled_kernels(kind):
    """The energies of a short range are those of the shaped kernels to the bit:
    the sums of a workgroup that holds all rows round differently."""
    prob = problem(kind)
    R = 32
    h0 = W.initial_fields(prob.n, R, seed=5, std=1.0)
    out = []
    for tiled in (False, True):
        s = solver(prob, R, kind, False)
        if tiled:
            s.set_tile(*s.tile())
        s.set_fields(h0)
        s.step(1)
        e = [s.energies()]
        s.run_until(s.t + 1)
        e.append(s.energies())
        out.append(np.array(e))
    assert np.array_equal(*out)


def test_no_marginal_copy_is_relied_on_after_a_callers_graph():
    """A caller's graph of steps moves the fields without the solver's
    knowledge; a short range after its replay starts from the moved fields."""
    prob = problem("rows 2")
    R = 8
    h0 = W.initial_fields(prob.n, R, seed=6, std=0.4)
    s = solver(prob, R, "rows 2", False)
    s.set_fields(h0)
    s.step(1)                          # a short range: row-tiled
    s.set_fields(h0)
    stream = torch.cuda.Stream()
    s2 = fem.Solver(prob, fem.default_params(replicas=R, steps=400), stream=stream)
    s2.set_fields(h0)
    s2.step(1)
    s2.set_fields(h0)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        s2.step(2)
    for k in (2, 30):
        ref = fem.Solver(prob, fem.default_params(replicas=R, steps=400))
        ref.set_tile(*TILE)
        ref.set_fields(h0)
        ref.step(2)
        h, m1, m2 = (np.frombuffer(ref.get_state()[-(3 * h0.nbytes + 8 * R):][i * h0.nbytes:(i + 1) * h0.nbytes],
                                   np.float32).reshape(h0.shape) for i in range(3))
        assert np.array_equal(h, ref.fields())
        s2.set_fields(h0)
        s2.step(1)                     # leaves a marginal copy of other fields behind
        s2.set_fields(h0)
        g.replay()
        stream.synchronize()
        assert np.array_equal(s2.fields(), h)
        s2.step(k)                     # from t = 0 as far as the solver knows
        ref.set_adam_state(h, m1, m2, 0)
        ref.step(k)
        assert np.array_equal(s2.fields(), ref.fields())


@pytest.mark.parametrize("kind", ["rows 2", "batch"])
def test_the_tuner_times_the_row_tiled_kernels(kind, tmp_path, monkeypatch):
    """A shape that is no candidate of the tuner, three rows per team, is taken
    from the cache, but not kept or written again by a tuning run; the solver's
    steps go on as if untuned, and long ones stay on one compute unit."""
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("FEM_TUNE_CACHE", str(cache))
    prob = problem(kind)
    R = 8
    h0 = W.initial_fields(prob.n, R, seed=7, std=0.4)
    s = solver(prob, R, kind, False)
    s.set_fields(h0)
    s.tune(trial_steps=1, use_cache=False)
    key = cache.read_text().split()[0]
    cache.write_text(f"{key} 1 4 3 0 8\n")
    assert s.tune(trial_steps=1, use_cache=True) == (1, 4, 3, 0, 8) == s.tile()
    s.step(5)
    tile = s.tune(trial_steps=2, use_cache=False)
    assert tile[2] != 3 and tile == s.tile()
    assert cache.read_text().splitlines()[-1].split() == [key] + [str(v) for v in tile]
    s.step(30)
    e = s.energies()
    out = []
    for tiled in (False, True):
        r = solver(prob, R, kind, tiled)
        r.set_fields(h0)
        r.step(5)
        r.step(30)
        out.append(r.energies())
        assert np.array_equal(r.fields(), s.fields())
    assert np.array_equal(e, out[0]) and not np.array_equal(e, out[1])


@pytest.mark.parametrize("kind", ["rows 2", "batch", "sat batch", "manip"])
def test_solvers_of_one_problem_share_its_tables(kind):
    """Solvers made by several threads at once, with other replica counts and
    schedules, stepping side by side after the problem and the solver that built
    the tables are gone."""
    prob = problem(kind)
    counts = [3, 8, 17, 32, 5, 64]
    h0 = [W.initial_fields(prob.n, R, seed=R, std=0.4) for R in counts]

    def run(k, tiled=False):
        s = solver(prob, counts[k], kind, tiled)
        s.set_fields(h0[k])
        return s

    with ThreadPoolExecutor(len(counts)) as pool:
        made = list(pool.map(run, range(len(counts))))
        ref = [run(k, tiled=True) for k in range(len(counts))]
        prob.close()
        for k in (0, 2):
            made[k].close()
        torch.cuda.synchronize()

        def go(k):
            out = []
            for n in (40, 33):
                made[k].step(n)
                out.append(made[k].fields())
            return out

        for k, got in zip((1, 3, 4, 5), pool.map(go, (1, 3, 4, 5))):
            for n, h in zip((40, 33), got):
                ref[k].step(n)
                assert np.array_equal(ref[k].fields(), h), k


@pytest.mark.parametrize("n,deg,weights,R,manip,resident", [
    (1000, 250, "pm1", 16, False, True), (1000, 250, "real", 16, False, False), (1000, 180, "real", 16, False, True),
    (2000, 100, "one", 16, False, False), (2000, 90, "one", 16, False, True), (2000, 100, "real", 64, False, True),
    (4000, 48, "pm1", 16, False, False), (4000, 48, "pm1", 64, False, True), (4000, 24, "pm1", 16, True, False),
    (4000, 24, "pm1", 64, True, True), (4000, 20, "real", 63, True, False), (4000, 20, "real", 64, True, True),
    (4000, 35, "pm1", 23, False, False), (4000, 35, "pm1", 24, False, True), (4000, 46, "pm1", 39, False, False), (4000, 46, "pm1", 40, False, True),
    (4000, 26, "real", 23, False, True), (4000, 32, "real", 23, False, False), (4000, 32, "real", 24, False, True)])
def test_entries_that_stream(n, deg, weights, R, manip, resident):
    """Long ranges with entries beyond LDS, on both sides of the rule: resident
    energies round otherwise than the shaped kernels' where a thread holds several
    rows; the fields are the same."""
    prob = graph(n, deg, weights)
    kw = {} if not manip else dict(gradient=fem.GRAD_MANIPULATED, energy_every=0)
    h0 = W.initial_fields(n, R, seed=8, std=1.0)
    out = []
    for tiled in (False, True):
        s = fem.Solver(prob, fem.default_params(replicas=R, steps=80, **kw), stream=torch.cuda.Stream())
        if tiled:
            s.set_tile(*s.tile())
        s.set_fields(h0)
        s.run_until(40)
        s.step(40)
        out.append((s.fields(), None if manip else np.array(s.energies())))
        s.close()
    assert np.array_equal(out[0][0], out[1][0])
    if not manip and (n > 1024 or not resident):
        assert np.array_equal(out[0][1], out[1][1]) != resident


def test_threads_that_need_different_amounts_of_lds():
    """Two problems run by the same kernel with 80 and 112 KB of LDS, stepped by
    two threads at once."""
    made = []
    for k, deg in enumerate((12, 20)):
        prob = graph(2000, deg)
        h0 = W.initial_fields(2000, 4, seed=9 + k, std=0.4)
        ref = solver(prob, 4, "maxcut", True)
        s = solver(prob, 4, "maxcut", False)
        for x in (s, ref):
            x.set_fields(h0)
        ref.step(400)
        made.append((s, ref.fields()))

    def go(k):
        for _ in range(50):
            made[k][0].step(8)
        return made[k][0].fields()

    with ThreadPoolExecutor(2) as pool:
        for (_, want), got in zip(made, pool.map(go, (0, 1))):
            assert np.array_equal(got, want)


def test_energy_sums_of_eight_rows_per_thread():
    """Equal fields in every row, one per replica: entropies that are sums of
    equal float32 terms.  Where a term's last two mantissa bits are zero, sums of
    up to four are exact in float32 (of five to eight they are not), and so is
    the entropy in double."""
    n, R = 8190, 256
    h = np.linspace(0.05, 2.5, R, dtype=np.float32)
    prob = fem.Problem.maxcut(n, [0], [1], [1.0])
    one = fem.Problem.maxcut(1, [], [])
    S = []
    for p, rows in ((prob, n), (one, 1)):
        s = fem.Solver(p, fem.default_params(replicas=R, steps=100, energy_every=100), stream=torch.cuda.Stream())
        s.set_fields(np.tile(h, (rows, 1)))
        s.step(40)
        S.append(s.energies()[1][0])
    term = S[1].astype(np.float32)
    assert np.array_equal(term.astype(np.float64), S[1])
    exact = (term.view(np.uint32) & 3) == 0
    assert exact.sum() > 30
    assert np.array_equal(S[0][exact], n * S[1][exact])
