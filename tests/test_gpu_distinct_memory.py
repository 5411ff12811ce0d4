"""The solve that handles every distinct instance once, around the batch (an instance per SIMD)
up to which every instance is solved as it is, and beyond, whatever the workspace holds
from other calls.  Integer work: every output must be equal."""

import numpy as np
import pytest

from distinct_calls import NAMES, side_by_side
from paper_2407_14843_amd import workloads as wl
from test_gpu_cost_solve import T  # noqa: F401

pytestmark = pytest.mark.gpu


def batch(oracle, idx, pool, n, seed, shared=False):
    """n instances of a pool, and the pool's answers for them."""
    rng = np.random.default_rng(seed)
    w = wl.workload(idx, pool)
    pick = rng.integers(0, pool, n)
    pick[: min(n, pool)] = rng.permutation(pool)[: min(n, pool)]
    want = [x[pick] for x in oracle.solve(w, threads=8)]
    return w.take(pick), want


def check(b, want, what):
    for name, g, x in zip(NAMES, b.results(), want):
        bad = np.nonzero((g != x).reshape(len(x), -1).any(axis=1))[0]
        assert bad.size == 0, f"{what}: {name} differs at {bad[:8]}"


@pytest.mark.parametrize("idx,pool,extra", [(1, 50, -1), (1, 50, 0), (1, 50, 1), (4, 300, 1), (2, 60, 512),
                                            (0, 1, 513), (1, 1200, 1025), (4, 90, 12000), (1, 2000, 6144 + 1)])
def test_whatever_the_workspace_holds(T, oracle, idx, pool, extra):
    import torch
    n = side_by_side() + extra
    w, want = batch(oracle, idx, pool, n, 50 + idx)
    b = T.DeviceBatch(w)
    b.solve_distinct()
    ws = b.memo_workspace
    fills = [lambda: ws.zero_(), lambda: ws.fill_(255), lambda: ws.fill_(0x11),
             lambda: ws.copy_(torch.randint(0, 256, ws.shape, dtype=torch.uint8, device=ws.device)),
             lambda: None]
    for k, fill in enumerate(fills):
        print(f"[case] workload {idx}, {n} instances of {pool}, filling {k}", flush=True)
        fill()
        for out in (b.status, b.cost, b.ticks, b.cfg):
            out.fill_(77)
        b.solve_distinct()
        check(b, want, f"filling {k}")


def test_inputs_that_change_under_the_same_workspace(T, oracle):
    """What calls before this one left, with the same instances at other places."""
    n = side_by_side() + 700
    rng = np.random.default_rng(4)
    w, want = batch(oracle, 1, 200, n, 9)
    b = T.DeviceBatch(w)
    b.solve_distinct()
    held = b.memo_workspace.clone()
    for k in range(4):
        order = rng.permutation(n)
        v = T.DeviceBatch(w.take(order))
        v.solve_distinct()
        v.memo_workspace.copy_(b.memo_workspace if k % 2 else held)
        v.solve_distinct()
        check(v, [x[order] for x in want], f"order {k}")


@pytest.mark.parametrize("n", [1, 7, 511, 512, 513])
def test_more_models_than_lanes(T, oracle, n):
    """The three stages, which take rates of zero instead of a list."""
    rng = np.random.default_rng(n)
    coef = wl._draw_coef(rng, (4, 65), a=(1000, 9000), k=(100, 1000), q=(0, 10), p=(1, 3), o=(1, 500))
    w = wl.Workload("models", wl.JOINT, 4, 65, 3, [1, 2, 3], 20, 1000, 900_000, False, coef,
                    rng.integers(1, 900, 4).astype(np.int32),
                    rng.integers(0, 900_001, 4).astype(np.int32))
    w = w.take(rng.integers(0, 4, n))
    want = oracle.solve(w, threads=8)
    b = T.DeviceBatch(w)
    b.solve_distinct()
    for fill in (0, 255):
        b.memo_workspace.fill_(fill)
        b.solve_distinct()
        check(b, want, f"{n} instances, filled with {fill}")
