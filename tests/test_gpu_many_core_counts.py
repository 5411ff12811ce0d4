"""GPU parity of every solve entry point with one batch size and thousands of core counts
per replica: the largest candidate indices with the fewest batch sizes to divide them by.
Whole numbers: no tolerance."""

import numpy as np
import pytest

from distinct_calls import distinct
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


def batch(n, n_stage, c_max, batch_sizes=(1,), slo=(100, 400), lam=(1, 4000)):
    """Models that need thousands of cores per replica to meet their objectives."""
    rng = np.random.default_rng([n_stage, c_max, len(batch_sizes)])
    coef = wl._draw_coef(rng, (n, n_stage), a=(1 << 19, 1 << 20), k=(0, 2000), q=(0, 1), p=(c_max // 2, c_max),
                         o=(1, 3))
    return wl.Workload("cores", wl.JOINT, n, n_stage, c_max, list(batch_sizes),
                       32767 // (n_stage * c_max), 1, slo[1], False, coef,
                       rng.integers(lam[0], lam[1] + 1, n).astype(np.int32),
                       rng.integers(slo[0], slo[1] + 1, n).astype(np.int32))


# (two models: the answer is thousands of cores above the least, past every window)
@pytest.mark.parametrize("n_stage,c_max,slo", [(1, 6000, (90, 250)), (1, 8192, (60, 400)),
                                               (2, 5000, (300, 900)), (2, 8192, (220, 600)),
                                               (4, 8191, (300, 1500))])
def test_joint_and_vertical(T, oracle, n_stage, c_max, slo):
    w = batch(48, n_stage, c_max, slo=slo)
    print(f"[case] {n_stage} models, {c_max} cores", flush=True)
    want = oracle.solve(w, threads=8)
    high = want[3][..., 0][want[0] == 0]
    assert (high > 4096).any(), "no answer takes an index beyond 4095"
    b = T.DeviceBatch(w)
    b.solve()
    same(b.results(), want)
    v = w.with_r_fixed(np.random.default_rng(1).integers(1, w.r_max + 1, (w.n_inst, n_stage)))
    b = T.DeviceBatch(v)
    b.solve()
    same(b.results(), oracle.solve(v, threads=8))


@pytest.mark.parametrize("batch_sizes", [(1,), (3,), (1, 2)])
def test_given_cores_and_the_rest(T, oracle, batch_sizes):
    c_max = 8192 // len(batch_sizes)
    # (a batch waits for its last request: rates and objectives that leave time for it)
    w = batch(40, 2, c_max, batch_sizes, (300, 1500), (1, 1500) if batch_sizes == (1,) else (3000, 12000))
    rng = np.random.default_rng(2)
    cores = rng.integers(c_max // 2, c_max + 1, (w.n_inst, 2)).astype(np.int32)
    cores[0] = c_max
    print(f"[case] given cores, batch sizes {batch_sizes}", flush=True)
    b = T.DeviceBatch(w)
    b.solve_horizontal(cores)
    want = oracle.solve(w, threads=8, c_fixed=cores)
    assert (want[0] == 0).any()
    same(b.results(), want)
    pred = (w.lam + rng.integers(0, 2, w.n_inst)).astype(np.int32)
    stable = b.check_stability(pred, cores)
    want = oracle.stability(w, pred, cores)
    assert (stable.cpu().numpy() == want[0]).all()
    same(b.results(), want[1:])
    b.solve_distinct()
    want = oracle.solve(w, threads=8)
    same(b.results(), want)
    distinct(T, w, want, sizes=("beyond",))
    v = w.with_r_fixed(np.ones((w.n_inst, 2), np.int32))
    v.lam = (v.lam * 5).astype(np.int32)
    b = T.DeviceBatch(v)
    b.solve_vertical_fallback()
    got, want = b.fallback_results(), oracle.vertical_fallback(v, threads=8)
    for k in want:
        assert (got[k] == want[k]).all(), k


def test_kept_results(T, oracle):
    """The calls that look at a workspace after a solve see the same configuration."""
    import torch
    w = batch(8, 1, 8000)
    b = T.DeviceBatch(w)
    b.solve()
    out = T.alloc_outputs(b.p, b.device)
    T.themis_stage_backtrack(b.p, *out, b.workspace)
    torch.cuda.synchronize()
    same(tuple(o.cpu().numpy() for o in out), oracle.solve(w, threads=4))
