"""GPU parity of the one-wavefront solve where its branches meet, and the calls that
look at the workspace after a solve.  Whole numbers: no tolerance."""

import numpy as np
import pytest

from cost_families import families, over_base
from paper_2407_14843_amd import workloads as wl

pytestmark = pytest.mark.gpu

NAMES = ("status", "cost", "ticks", "cfg")


@pytest.fixture(scope="module")
def T():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2407_14843_amd import themis
    themis.lib()
    return themis


def same(got, want):
    for n, g, x in zip(NAMES, got, want):
        bad = np.nonzero((g != x).reshape(len(x), -1).any(axis=1))[0]
        assert bad.size == 0, f"{n} differs at {bad[:8]}: got {g[bad[:2]]}, want {x[bad[:2]]}"


# A wavefront has the more LDS the fewer instances there are: the most at 240, the least at
# 7200 (the same 240 again and again).  test_gpu_steps_met.py has which steps that takes.
@pytest.mark.parametrize("n", [1, 240, 7200])
@pytest.mark.parametrize("name", list(families(1)))
def test_windows(T, oracle, name, n):
    w = families(min(n, 240))[name]
    again = np.arange(n) % w.n_inst
    want = tuple(x[again] for x in oracle.solve(w, threads=8))
    w = w.take(again)
    print(f"[case] {name} N={n}", flush=True)
    b = T.DeviceBatch(w)
    b.solve()
    same(b.results(), want)


def test_windows_are_met(oracle):
    """The answers of the batches above lie anywhere over the least cost: at it, inside the
    windows of 16 and of 64 cells, and hundreds and thousands of cores beyond."""
    x = np.concatenate([over_base(w, oracle, oracle.solve(w, threads=8))
                        for w in families(240).values()])
    for lo, hi in ((0, 0), (1, 15), (16, 63), (64, 255), (256, 1023), (1024, 32767)):
        assert ((x >= lo) & (x <= hi)).any(), (lo, hi)


def test_many_models_in_every_entry_point(T, oracle):
    """More models than lanes: the passes of the three stages behind every entry point."""
    rng = np.random.default_rng(66)
    n, S = 33, 66
    coef = wl._draw_coef(rng, (n, S), a=(1000, 9000), k=(100, 1000), q=(0, 10), p=(1, 3), o=(1, 500))
    w = wl.Workload("models", wl.JOINT, n, S, 3, [1, 2, 4], 20, 1000, 900_000, False, coef,
                    rng.integers(1, 900, n).astype(np.int32),
                    rng.integers(0, 900_001, n).astype(np.int32))
    w = w.take(np.arange(2 * n) % n)
    b = T.DeviceBatch(w)
    b.solve_distinct()
    same(b.results(), oracle.solve(w, threads=8))
    pred = np.where(np.arange(2 * n) % 3 == 0, w.lam + 1, w.lam).astype(np.int32)
    stable = b.check_stability(pred)
    want = oracle.stability(w, pred)
    assert (stable.cpu().numpy() == want[0]).all()
    same(b.results(), want[1:])
    v = w.with_r_fixed(rng.integers(1, 4, (w.n_inst, S)))
    b = T.DeviceBatch(v)
    b.solve_vertical_fallback()
    got, want = b.fallback_results(), oracle.vertical_fallback(v, threads=8)
    for k in want:
        assert (got[k] == want[k]).all(), k


@pytest.mark.parametrize("n_stage", [1, 2, 63, 64, 65])
def test_model_counts(T, oracle, n_stage):
    """A lane per model up to 64; more take the three stages."""
    rng = np.random.default_rng(n_stage)
    n = 37
    coef = wl._draw_coef(rng, (n, n_stage), a=(1000, 9000), k=(100, 1000), q=(0, 10), p=(1, 3),
                         o=(1, 500))
    w = wl.Workload("models", wl.JOINT, n, n_stage, 3, [1, 2, 3], 20, 1000, 900_000, False, coef,
                    rng.integers(1, 900, n).astype(np.int32),
                    rng.integers(0, 900_001, n).astype(np.int32))
    b = T.DeviceBatch(w)
    b.solve()
    want = oracle.solve(w, threads=8)
    same(b.results(), want)
    assert (want[0] == 0).any()


def staged(T, w, prune):
    """tables and counts after the candidate stage"""
    b = T.DeviceBatch(w, prune=prune)
    T.themis_stage_candidates(b.p, b.coef, b.lam, b.slo_us, b.r_fixed, b.workspace)
    return inspect(T, b)


def inspect(T, b):
    import torch
    shape = (b.p.n_inst, b.p.n_stage, b.w.n_cand)
    lt = torch.empty(shape, dtype=torch.int32, device=b.device)
    co = torch.empty(shape, dtype=torch.int32, device=b.device)
    cnt = torch.empty(3, dtype=torch.int64, device=b.device)
    T.themis_export_candidates(b.p, b.workspace, lt, co)
    T.themis_count_relaxations(b.p, b.workspace, cnt)
    torch.cuda.synchronize()
    return lt.cpu().numpy(), co.cpu().numpy(), cnt.cpu().numpy()


def backtrack(T, b):
    out = T.alloc_outputs(b.p, b.device)
    T.themis_stage_backtrack(b.p, *out, b.workspace)
    return tuple(o.cpu().numpy() for o in out)


@pytest.mark.parametrize("prune", [0, 1])
@pytest.mark.parametrize("idx,n", [(0, 64), (2, 70), (3, 1100), (4, 1030)])
def test_workspace_after_a_solve(T, oracle, idx, n, prune):
    """Tables, counts and results can be had from the workspace after a solve as after
    the stage calls, in any order, and the stage calls work on it afterwards."""
    w = wl.workload(idx, n)
    w.lam[3] = 0  # an invalid instance
    print(f"[case] inspect workload {idx} N={n} prune={prune}", flush=True)
    lt_w, co_w, cnt_w = staged(T, w, prune)
    want = oracle.solve(w, threads=8)
    b = T.DeviceBatch(w, prune=prune)
    for order in ("tables first", "results first"):
        b.solve()
        same(b.results(), want)
        if order == "results first":
            same(backtrack(T, b), want)
        for _ in range(2):
            lt, co, cnt = inspect(T, b)
            assert (lt == lt_w).all() and (co == co_w).all() and (cnt == cnt_w).all()
            T.themis_stage_minplus(b.p, b.workspace)  # nothing is listed: no effect
            same(backtrack(T, b), want)
    T.themis_stage_candidates(b.p, b.coef, b.lam, b.slo_us, b.r_fixed, b.workspace)
    T.themis_stage_minplus(b.p, b.workspace)
    same(backtrack(T, b), want)


def test_workspace_after_a_horizontal_solve(T, oracle):
    w = wl.workload(1, 50)
    rng = np.random.default_rng(1)
    cores = rng.integers(1, w.c_max + 1, (w.n_inst, w.n_stage)).astype(np.int32)
    b = T.DeviceBatch(w)
    b.solve_horizontal(cores)
    want = oracle.solve(w, threads=8, c_fixed=cores)
    same(b.results(), want)
    lt, co, _ = inspect(T, b)
    lt_o, co_o, _ = oracle.candidates(w)
    c = np.arange(w.n_cand) // len(w.batch_sizes) + 1
    mine = c[None, None] == cores[..., None]
    assert (lt == np.where(mine, lt_o, -1)).all()
    assert (co == np.where(mine & (lt_o >= 0), co_o, -1)).all()
    same(backtrack(T, b), want)


@pytest.mark.parametrize("idx,n", [(2, 60), (4, 9000)])
def test_fallback_and_stability_in_one_wavefront(T, oracle, idx, n):
    """The multi-solve entry points on one launch and on two, with overload, rates equal to
    the prediction and a prediction out of range."""
    w = wl.workload(idx, n)
    rng = np.random.default_rng(idx)
    if idx == 4:
        w = w.with_r_fixed(rng.integers(1, 5, (w.n_inst, w.n_stage)))
    w.lam = np.minimum(w.lam.astype(np.int64) * rng.integers(1, 6, n), 1 << 20).astype(np.int32)
    w.lam[1] = -5
    b = T.DeviceBatch(w)
    b.solve_vertical_fallback()
    got, want = b.fallback_results(), oracle.vertical_fallback(w, threads=8)
    for k in want:
        assert (got[k] == want[k]).all(), k
    assert ((want["lambda_v"] > 0) & (want["lambda_v"] < w.lam)).any()  # searched and split
    pred = np.where(rng.random(n) < 0.5, w.lam, w.lam + rng.integers(-2, 30, n)).astype(np.int32)
    pred[2] = 0
    stable = b.check_stability(pred)
    want = oracle.stability(w, pred)
    assert (stable.cpu().numpy() == want[0]).all()
    same(b.results(), want[1:])
    assert 0 < want[0].mean() < 1


def test_workspace_after_multi_solves(T, oracle):
    """After a multi-solve call the workspace shows its last solve: instances that one was
    not given have no tables and read as invalid."""
    w = wl.workload(4, 1100)
    w = w.take(np.arange(1100) % 400)
    b = T.DeviceBatch(w)
    b.workspace = __import__("torch").empty(T.memo_workspace_bytes(b.p), dtype=b.workspace.dtype,
                                            device=b.device)
    b.memo_workspace = b.workspace
    b.solve_distinct()
    want = oracle.solve(w, threads=8)
    same(b.results(), want)
    lt, _, _ = inspect(T, b)
    lt_o, _, _ = oracle.candidates(w)
    solved_here = (lt >= 0).any(axis=(1, 2))
    assert 0 < solved_here.sum() < w.n_inst
    assert (lt[solved_here] == lt_o[solved_here]).all()
    got = backtrack(T, b)
    same(tuple(g[solved_here] for g in got), tuple(x[solved_here] for x in want))
    assert (got[0][~solved_here] == 2).all() and (got[3][~solved_here] == 0).all()
