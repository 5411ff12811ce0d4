"""Which step of the one-wavefront solve finds the answers of which batch: the batches below
reach every step and every place of its rows, with the answers the checker gives.  The step
is kept with the results (solve_steps.py); a batch that no longer reaches the step it is here
for fails.  Whole numbers: no tolerance."""

import numpy as np
import pytest

from cost_families import families, family, over_base
from distinct_calls import distinct
from paper_2407_14843_amd import workloads as wl
from solve_steps import STEPS, steps_by_rule, steps_of
from test_gpu_cost_solve import T, same  # noqa: F401

pytestmark = pytest.mark.gpu


def solved(T, oracle, w, n=None):
    """Solves w (its instances again and again up to n), checks it and returns the steps."""
    want = oracle.solve(w, threads=8)
    again = np.arange(n or w.n_inst) % w.n_inst
    b = T.DeviceBatch(w.take(again))
    b.solve()
    same(b.results(), tuple(x[again] for x in want))
    step = steps_of(b.p, b.workspace)
    assert ((step >= 0) == (want[0][again] == 0)).all()
    print("[steps]", {s: int((step == k).sum()) for k, s in enumerate(STEPS) if (step == k).any()},
          flush=True)
    return step[:w.n_inst], want


def long_pipelines(S, n):
    """Sixteen and more models: a wavefront's LDS has little room for lists and rows"""
    return family(3, n, S, 8, [1, 2, 4, 8], 32767 // (S * 8) // 2, 500, 2_000_000, (10, 2000))


def dense(n, tick, slo, lam=(10, 20_000)):
    """Thousands of candidates per model: more than any list has room for"""
    return family(3, n, 3, 512, list(range(1, 17)), 20, tick, slo, lam)


# at 240 instances a wavefront has the most LDS, at 7200 the least
@pytest.mark.parametrize("n", [240, 7200])
@pytest.mark.parametrize("name,steps", [
    ("three models", "A,B,C,G trial"), ("four models", "A,C,G trial"),
    ("eight models", "A,B,C,G trial"), ("ten models, replicas given", "A,B,C,G trial"),
    ("many cores", "A,B,C,G trial"), ("long lists", "B,C,G trial"), ("one model", "A")])
def test_families(T, oracle, name, steps, n):
    step, _ = solved(T, oracle, families(240)[name], n)
    met = {STEPS[k] for k in np.unique(step[step >= 0])}
    for s in steps.split(","):
        assert any(m.startswith(s) for m in met), s


@pytest.mark.parametrize("w,n,steps", [
    (lambda: long_pipelines(32, 96), 96, "G LDS"),
    (lambda: long_pipelines(32, 96), 4100, "G HBM"),
    (lambda: long_pipelines(64, 64), 64, "G LDS"),
    (lambda: long_pipelines(64, 64), 2100, "G HBM"),
    (lambda: dense(96, 5, 30_000), 96, "C,G trial"),
    (lambda: dense(96, 5, 30_000), 4200, "C,G trial"),
    (lambda: dense(64, 100, 200_000), 64, "A,B,G trial")])
def test_little_room_and_many_candidates(T, oracle, w, n, steps):
    step, _ = solved(T, oracle, w(), n)
    met = {STEPS[k] for k in np.unique(step[step >= 0])}
    for s in steps.split(","):
        assert any(m.startswith(s) for m in met), s


# Lists that no wavefront of a full compute unit has room for, however they are cut (of some
# thousand instances drawn one each).  The windows in LDS are tried first, without success.
@pytest.mark.parametrize("w,which,steps", [
    (lambda: family(5, 3000, 4, 512, list(range(1, 17)), 15, 2, 20_000, (1000, 60_000)),
     [914, 964, 1994], "W HBM,D"),
    (lambda: family(6, 2000, 8, 256, list(range(1, 17)), 15, 2, 30_000, (1000, 60_000)),
     [167, 375, 734], "W HBM,D"),
    (lambda: family(3, 4096, 3, 512, list(range(1, 17)), 20, 5, 30_000, (10, 20_000)),
     [2714, 3546], "D")])
def test_last_resorts(T, oracle, w, which, steps):
    step, _ = solved(T, oracle, w().take(which), 7200)
    met = {STEPS[k] for k in np.unique(step[step >= 0])}
    for s in steps.split(","):
        assert any(m.startswith(s) for m in met), s


@pytest.mark.parametrize("x", [14, 15, 16, 17, 62, 63, 64, 65])
def test_window_edges(T, oracle, x):
    """Answers right at the edges of the windows of 16 and 64 cells."""
    w = families(6000)["three models"]
    status, cost, ticks, cfg = oracle.solve(w, threads=8)
    at = np.nonzero(status == 0)[0]
    over = over_base(w, oracle, (status, cost))
    pick = at[over == x]
    assert pick.size, "no such instance"
    step, want = solved(T, oracle, w.take(pick))
    rule = steps_by_rule(w.take(pick), oracle, want)
    assert all(r in ("B8", "B16", "C") if x < 64 else r == "" for r in rule), rule
    for k, r in zip(step, rule):
        assert STEPS[k] == r if r else STEPS[k].startswith("G"), (STEPS[k], r)


# The forms in which the steps after B are compiled or fed: queue models, Eq. 1's delta, cores
# given or one for all, replicas given, rates of the fallback and the stability test, lists of
# instances.  (Short objectives send most instances past step B.)
@pytest.mark.parametrize("queue", [0, 1, 2])
@pytest.mark.parametrize("delta", [False, True])
@pytest.mark.parametrize("name", ["eight models", "long lists", "many cores"])
def test_every_form(T, oracle, name, queue, delta):
    w = families(240)[name].take(np.arange(48))
    rng = np.random.default_rng([queue, delta])
    w = w.with_model(queue, rng.integers(0, 300, w.coef.shape[:-1]) if delta else None)
    print(f"[case] {name} queue {queue} delta {delta}", flush=True)
    solved(T, oracle, w)
    b = T.DeviceBatch(w)
    b.solve_distinct()
    want = oracle.solve(w, threads=8)
    same(b.results(), want)
    distinct(T, w, want, sizes=("beyond",))
    for cores in (None, rng.integers(1, w.c_max + 1, (w.n_inst, w.n_stage)).astype(np.int32)):
        b.solve_horizontal(cores)
        same(b.results(), oracle.solve(w, threads=8, c_fixed=cores if cores is not None
                                       else np.ones((w.n_inst, w.n_stage), np.int32)))
        pred = np.minimum(w.lam + rng.integers(0, 3, w.n_inst), 1 << 20).astype(np.int32)
        stable = b.check_stability(pred, cores)
        want = oracle.stability(w, pred, cores)
        assert (stable.cpu().numpy() == want[0]).all()
        same(b.results(), want[1:])
    v = w.with_r_fixed(rng.integers(1, min(w.r_max, 200) + 1, (w.n_inst, w.n_stage)))
    solved(T, oracle, v)
    b = T.DeviceBatch(v)
    b.solve_vertical_fallback()
    got, want = b.fallback_results(), oracle.vertical_fallback(v, threads=8)
    for k in want:
        assert (got[k] == want[k]).all(), k
