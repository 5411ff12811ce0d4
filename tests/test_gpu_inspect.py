"""The calls that look at a workspace (tables, counts, kept results) only read it: its
bytes stay as they were, and calls on several streams at once see the same.  Tables and
counts after a whole solve are those of the candidate stage.  Whole numbers: no
tolerance."""

import numpy as np
import pytest

from paper_2407_14843_amd import workloads as wl
from test_gpu_cost_solve import NAMES, T, inspect, same, staged  # noqa: F401

pytestmark = pytest.mark.gpu


def buffers(T, b, torch):
    shape = (b.p.n_inst, b.p.n_stage, b.w.n_cand)
    new = lambda: torch.empty(shape, dtype=torch.int32, device=b.device)
    return new(), new(), torch.empty(3, dtype=torch.int64, device=b.device), T.alloc_outputs(b.p, b.device)


def look(T, b, buf, stream=None):
    T.themis_export_candidates(b.p, b.workspace, buf[0], buf[1], stream)
    T.themis_count_relaxations(b.p, b.workspace, buf[2], stream)
    T.themis_stage_backtrack(b.p, *buf[3], b.workspace, stream)


@pytest.mark.parametrize("how", ["solve", "stages"])
@pytest.mark.parametrize("prune", [0, 1, 2, 3])
def test_only_read_and_at_once(T, oracle, prune, how):
    import torch
    w = wl.workload(1, 1500)
    w.lam[7] = 0  # an invalid instance
    lt, co, cnt = staged(T, w, prune)
    want = oracle.solve(w, threads=8)
    b = T.DeviceBatch(w, prune=prune)
    b.workspace.zero_()
    if how == "solve":
        b.solve()
    else:
        T.themis_stage_candidates(b.p, b.coef, b.lam, b.slo_us, b.r_fixed, b.workspace)
        T.themis_stage_minplus(b.p, b.workspace)
    before = b.workspace.clone()
    streams = [torch.cuda.Stream() for _ in range(3)]
    bufs = [buffers(T, b, torch) for _ in streams]
    torch.cuda.synchronize()
    for _ in range(4):
        for st, buf in zip(streams, bufs):
            look(T, b, buf, st)
    torch.cuda.synchronize()
    assert torch.equal(b.workspace, before)
    for buf in bufs:
        for got, x in zip(buf[:3], (lt, co, cnt)):
            assert (got.cpu().numpy() == x).all()
        same(tuple(o.cpu().numpy() for o in buf[3]), want)


# one model and one candidate; rows cut by the most cores, by one batch size, by the
# largest table; costs that share a bin when pruned; rows longer than 16384 cells
@pytest.mark.parametrize("prune", [0, 1, 2])
@pytest.mark.parametrize("shape", [(70, 1, 1, [1], 1, 1000, 100_000), (33, 3, 7, [2, 3, 5], 30, 500, 400_000),
                                   (20, 2, 512, list(range(1, 17)), 30, 20, 300_000),
                                   (9, 64, 4, [1, 8], 100, 100, 3_000_000),
                                   (12, 2, 3, [1, 2, 4], 5000, 250, 500_000)])
@pytest.mark.parametrize("queue,delta,shared", [(0, False, False), (1, True, True), (2, False, True)])
def test_tables_after_a_solve(T, shape, prune, queue, delta, shared):
    n, S, c_max, batch_sizes, r_max, tick, slo = shape
    rng = np.random.default_rng([n, S, queue])
    coef = wl._draw_coef(rng, (S,) if shared else (n, S), a=(1000, 30000), k=(100, 3000), q=(0, 20),
                         p=(1, c_max), o=(1, 500))
    w = wl.Workload("inspect", wl.JOINT, n, S, c_max, batch_sizes, r_max, tick, slo, shared, coef,
                    rng.integers(1, 20_000, n).astype(np.int32),
                    rng.integers(0, slo + 1, n).astype(np.int32))
    w = w.with_model(queue, rng.integers(0, 300, coef.shape[:-1]) if delta else None)
    w.lam[n // 2] = -1
    print(f"[case] inspect {shape} queue {queue} prune {prune}", flush=True)
    for x in (w, w.with_r_fixed(rng.integers(1, min(r_max, 9) + 1, (n, S)))):
        tables = staged(T, x, prune)
        b = T.DeviceBatch(x, prune=prune)
        b.solve()
        for got, want in zip(inspect(T, b), tables):
            assert (got == want).all()
