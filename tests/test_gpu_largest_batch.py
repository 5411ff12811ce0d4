"""A batch of more instances than one launch with a wavefront each can have.  Whole
numbers: no tolerance."""

import numpy as np
import pytest

from paper_2407_14843_amd import workloads as wl

pytestmark = pytest.mark.gpu


def test_more_instances_than_a_launch_takes(oracle):
    """2^26 + 77 instances of one small model (25 GB of workspace), a pattern of 997 of them
    again and again, against the pattern's answers: the joint solve, what it keeps, and the
    stability test."""
    import torch
    from paper_2407_14843_amd import themis as T
    period, n, dev = 997, (1 << 26) + 77, "cuda:0"
    rng = np.random.default_rng(26)
    coef = wl._draw_coef(rng, (1,), a=(2000, 20000), k=(100, 1000), q=(0, 10), p=(1, 2), o=(1, 500))
    w = wl.Workload("largest", wl.JOINT, period, 1, 2, [1, 4], 8, 1000, 100_000, True, coef,
                    rng.integers(0, 900, period).astype(np.int32),
                    rng.integers(0, 100_001, period).astype(np.int32))
    w.lam[5::100] = 0  # invalid
    want = oracle.solve(w, threads=8)
    assert all((want[0] == s).any() for s in (0, 1, 2))
    pred = (w.lam + rng.integers(0, 40, period)).astype(np.int32)
    want_stable = oracle.stability(w, pred)

    at = torch.arange(n, device=dev) % period
    spread = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)[at]
    p = T.make_problem(n, 1, w.c_max, w.batch_sizes, w.r_max, w.tick_us, w.slo_max_us, True)
    lam, slo, lam_pred = spread(w.lam), spread(w.slo_us), spread(pred)
    coef_d = torch.from_numpy(w.coef).to(dev)
    ws = torch.empty(T.stability_workspace_bytes(p), dtype=torch.uint8, device=dev)
    out, stable = T.alloc_outputs(p, dev), torch.empty(n, dtype=torch.int32, device=dev)

    def check(what, got, expected):
        for k, (g, x) in enumerate(zip(got, expected)):
            assert torch.equal(g, spread(x.astype(np.int32))), (what, k)

    print(f"[case] {n} instances, joint", flush=True)
    T.themis_solve_joint(p, coef_d, lam, slo, *out, ws)
    check("joint", out, want)
    for o in out:
        o.fill_(-7)
    print("[case] what it keeps", flush=True)
    T.themis_stage_backtrack(p, *out, ws)
    check("kept", out, want)
    print("[case] stability", flush=True)
    T.themis_check_stability(p, coef_d, lam, lam_pred, slo, None, stable, *out, ws)
    check("stability", (stable,) + out, want_stable)
