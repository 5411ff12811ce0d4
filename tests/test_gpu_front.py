"""The start of the one-wavefront solve (csrc/cost_front.h) at the sizes where its branches
meet: every way the (model, batch size) pairs lie in a wavefront, answers at the edges of the
windows of four, eight and sixteen cells, and products beyond 2^42.  Whole numbers, so the
oracle's answers word for word: no tolerance."""

import numpy as np
import pytest

from cost_families import families, family, over_base
from distinct_calls import distinct
from paper_2407_14843_amd import workloads as wl
from solve_steps import STEPS, steps_by_rule, steps_of
from test_gpu_cost_solve import T, same  # noqa: F401

pytestmark = pytest.mark.gpu


def every_call(T, oracle, w, r_most):
    """Each entry point on w, against the oracle."""
    rng = np.random.default_rng(w.n_stage)
    b = T.DeviceBatch(w)
    b.solve()
    want = oracle.solve(w, threads=8)
    same(b.results(), want)
    b.solve_distinct()
    same(b.results(), want)
    distinct(T, w, want, sizes=("beyond",))
    cores = rng.integers(1, w.c_max + 1, (w.n_inst, w.n_stage)).astype(np.int32)
    b.solve_horizontal(cores)
    same(b.results(), oracle.solve(w, threads=8, c_fixed=cores))
    pred = np.minimum(w.lam + rng.integers(0, 3, w.n_inst), 1 << 20).astype(np.int32)
    stable = b.check_stability(pred)
    flags = oracle.stability(w, pred)
    assert (stable.cpu().numpy() == flags[0]).all()
    same(b.results(), flags[1:])
    v = w.with_r_fixed(rng.integers(1, r_most + 1, (w.n_inst, w.n_stage)))
    b = T.DeviceBatch(v)
    b.solve()
    same(b.results(), oracle.solve(v, threads=8))
    b.solve_vertical_fallback()
    got, fell = b.fallback_results(), oracle.vertical_fallback(v, threads=8)
    for k in fell:
        assert (got[k] == fell[k]).all(), k
    return want


# lanes per model 4, 8 and 16, the fewest and the most models and batch sizes that fit; pairs
# that fit only without gaps; more of them than lanes, in turns with gaps and without, and
# (33 x 2) in rounds of models
@pytest.mark.parametrize("S,n_batch", [
    (1, 1), (16, 4), (3, 3), (8, 8), (8, 5), (1, 16), (4, 16), (4, 9),
    (10, 6), (12, 5), (7, 9), (9, 7), (5, 12), (32, 2),
    (17, 4), (9, 8), (7, 12), (5, 16), (33, 2), (9, 9), (10, 10)])
@pytest.mark.parametrize("queue", [0, 1, 2])
def test_layouts(T, oracle, S, n_batch, queue):
    r_max = min(40, 32767 // (S * 7))
    w = family([S, n_batch], 96, S, 7, list(range(1, n_batch + 1)), r_max, 250, S * 60_000, (10, 900))
    w = w.with_model(queue, None)
    print(f"[case] {S} models, {n_batch} batch sizes, queue {queue}", flush=True)
    want = every_call(T, oracle, w, min(r_max, 6))
    assert (want[0] == 0).any()


@pytest.mark.parametrize("kind", ["derived", "given", "one core"])
def test_window_edges(T, oracle, kind):
    """Answers 0 to 17 over the least cost, all in one batch and each in one of its own, and the
    step that finds each of them."""
    w = {"derived": lambda: family(22, 4000, 6, 16, [1, 2, 4, 8, 16], 30, 250, 500_000, (10, 900)),
         "given": lambda: family(21, 4000, 6, 16, [1, 2, 4, 8, 16], 5, 250, 700_000, (10, 400), r_fixed=5),
         "one core": lambda: families(4000)["three models"]}[kind]()
    want = oracle.solve(w, threads=8)
    at = np.nonzero(want[0] == 0)[0]
    over = over_base(w, oracle, want)
    picks = [at[over == x][:40] for x in (0, 1, 3, 4, 5, 7, 8, 9, 15, 16, 17)]
    assert sum(p.size > 0 for p in picks) >= 9, [p.size for p in picks]
    met = set()
    for pick in picks + [np.concatenate(picks)]:
        if pick.size:
            v, x = w.take(pick), tuple(x[pick] for x in want)
            b = T.DeviceBatch(v)
            b.solve()
            same(b.results(), x)
            steps = np.array(STEPS)[steps_of(b.p, b.workspace)]
            rule = steps_by_rule(v, oracle, x)
            assert (steps == rule).all(), list(zip(steps, rule))
            met |= {(s, n) for s, n in zip(steps, over_base(v, oracle, x).tolist())}
    # each window up to its last cells, and step C where it found what step B was not asked for
    if kind == "one core":
        assert {("B8", 7), ("B16", 8), ("B16", 15), ("C", 16)} <= met, sorted(met)
        assert not any(s == "C" and n < 16 for s, n in met), sorted(met)
    else:
        assert {("B8", 7), ("B16", 15), ("B16", 8), ("C", 16)} <= met, sorted(met)
        assert any(s == "C" and n < 16 for s, n in met), sorted(met)


@pytest.mark.parametrize("S,n_batch", [(4, 7), (8, 8), (7, 9), (9, 9)])
def test_one_core_count(T, oracle, S, n_batch):
    """One candidate per model and batch size: one table for all windows."""
    rng = np.random.default_rng([S, n_batch])
    w = family([S, n_batch, 7], 600, S, 7, list(range(1, n_batch + 1)), 32767 // (S * 7), 250,
               S * 60_000, (10, 5000))
    for cores in (np.ones((w.n_inst, S), np.int32), rng.integers(1, 8, (w.n_inst, S)).astype(np.int32)):
        want = oracle.solve(w, threads=8, c_fixed=cores)
        b = T.DeviceBatch(w)
        b.solve_horizontal(cores)
        same(b.results(), want)
        rule = steps_by_rule(w, oracle, want, cores)
        steps = np.array(STEPS + ("",))[steps_of(b.p, b.workspace)]
        assert ((steps == rule) | (rule == "")).all(), list(zip(steps, rule))
        assert {"A", "B8", "B16", "C"} <= set(rule), set(rule)


@pytest.mark.parametrize("n_batch,queue", [(7, 0), (13, 0), (7, 2)])
def test_products_beyond_42_bits(T, oracle, n_batch, queue):
    """Rates times objectives on both sides of 2^42."""
    w = family(9, 300, 3, 1, [2 ** j if n_batch == 7 else j + 1 for j in range(n_batch)], 10_000,
               1000, 30_000_000, (50_000, 1_000_000)).with_model(queue, None)
    large = w.lam.astype(np.int64) * w.slo_us >= 1 << 42
    assert large.any() and not large.all()
    print(f"[case] beyond 2^42, three models, {n_batch} batch sizes, queue {queue}", flush=True)
    want = every_call(T, oracle, w, 10_000)
    assert (want[0][large] == 0).any()


# turns without gaps, more than eight models; rounds of ten, seven and twelve models
@pytest.mark.parametrize("S,n_batch,c_max,queue", [(10, 10, 1, 0), (17, 5, 1, 0), (17, 5, 1, 2), (9, 9, 2, 0),
                                                   (33, 6, 1, 2), (23, 9, 1, 0), (33, 5, 1, 0)])
def test_products_beyond_42_bits_in_rounds(T, oracle, S, n_batch, c_max, queue):
    """Answers of every window at rates times objectives beyond 2^42, with more pairs than lanes."""
    rng, n = np.random.default_rng([42, S, n_batch]), 300
    coef = wl._draw_coef(rng, (n, S), a=(1000, 40000), k=(100, 700), q=(0, 0), p=(1, c_max), o=(1, 2000))
    sizes = sorted({int(x) for x in np.rint(np.geomspace(2, 1024, n_batch))})
    r_max = 32767 // (S * c_max)
    w = wl.Workload("large", wl.JOINT, n, S, c_max, sizes, r_max, 1000, 30_000_000, False, coef,
                    rng.integers(100_000, 1_048_577, n).astype(np.int32),
                    rng.integers(1_000_000, 30_000_000, n).astype(np.int32)).with_model(queue, None)
    large = w.lam.astype(np.int64) * w.slo_us >= 1 << 42
    print(f"[case] beyond 2^42, {S} models, {n_batch} batch sizes, queue {queue}", flush=True)
    want = every_call(T, oracle, w, r_max)
    met = set(steps_by_rule(w, oracle, want)[large])
    assert {"A", "B16", "C"} <= met, met


@pytest.mark.parametrize("S,n_batch", [(8, 8), (16, 4), (4, 16), (7, 9), (9, 9)])
def test_cores_handed_on(T, oracle, S, n_batch):
    """The cores of the vertical part, found by any step and so left behind by any lane, are
    those of the new instances."""
    w = family([S, n_batch, 3], 400, S, 7, list(range(1, n_batch + 1)), min(40, 32767 // (S * 7)),
               250, S * 60_000, (10, 2500), r_fixed=6)
    want = oracle.vertical_fallback(w, threads=8)
    at = (want["lambda_v"] > 0) & (want["lambda_v"] < w.lam) & (want["status_h"] == 0)
    kept = w.take(np.arange(w.n_inst))
    kept.lam = np.maximum(want["lambda_v"], 1).astype(np.int32)
    met = set(steps_by_rule(kept, oracle, (want["status"], want["cost"]))[at])
    assert {"A", "B8", "B16", "C"} <= met, met
    cores = want["cfg"][at][:, :, 0]
    assert (cores.min(axis=1) < cores.max(axis=1)).mean() > 0.5
    print(f"[case] fallback {S} models, {n_batch} batch sizes", flush=True)
    b = T.DeviceBatch(w)
    b.solve_vertical_fallback()
    got = b.fallback_results()
    for k in want:
        assert (got[k] == want[k]).all(), k
