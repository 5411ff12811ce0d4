"""GPU parity of the three stage calls (candidate tables, recurrence over the budget,
selection and reconstruction), which the whole-solve entry points do not go through:
every workload, every form of the recurrence, rows around the edges of its tiles, random
options.  Whole numbers: no tolerance."""

import numpy as np
import pytest

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


def by_stages(T, w, prune):
    b = T.DeviceBatch(w, prune=prune)
    T.themis_stage_candidates(b.p, b.coef, b.lam, b.slo_us, b.r_fixed, b.workspace)
    T.themis_stage_minplus(b.p, b.workspace)
    T.themis_stage_backtrack(b.p, b.status, b.cost, b.ticks, b.cfg, b.workspace)
    return b.results()


# sizes on both sides of one workgroup's input check, of the small-batch geometry and,
# for workload 3, of the second launch of its recurrence
@pytest.mark.parametrize("prune", [0, 1, 2, 3])
@pytest.mark.parametrize("idx,n", [(0, 64), (1, 1500), (2, 200), (3, 120), (4, 1300)])
def test_workloads(T, oracle, idx, n, prune):
    w = wl.workload(idx, n)
    print(f"[case] stages, workload {idx} N={n} prune={prune}", flush=True)
    same(by_stages(T, w, prune), oracle.solve(w, threads=8))


@pytest.mark.parametrize("prune", [0, 1])
def test_many_instances(T, prune):
    """The launch geometries of a large batch, against the whole solve."""
    w = wl.workload(3, 24000)
    b = T.DeviceBatch(w)
    b.solve()
    same(by_stages(T, w, prune), b.results())


@pytest.mark.parametrize("cells", [1, 2, 127, 128, 129, 511, 512, 513, 1023, 1024, 1025, 8191,
                                   8192, 8193, 16383, 16384, 16385, 16386, 32767, 32768])
def test_row_lengths(T, oracle, cells):
    rng = np.random.default_rng(cells)
    n, S, tick = 4, 3, 100
    coef = wl._draw_coef(rng, (n, S), a=(2000, 60000), k=(500, 5000), q=(0, 50), p=(1, 8),
                         o=(100, 1000))
    slo = (cells - 1) * tick
    w = wl.Workload("rows", wl.JOINT, n, S, 8, [1, 2, 4, 8, 16], 8, tick, slo, False, coef,
                    rng.integers(10, 400, n).astype(np.int32), np.full(n, slo, np.int32))
    want = oracle.solve(w, threads=4)
    for prune in range(4):
        same(by_stages(T, w, prune), want)


def test_random_options(T, oracle):
    rng = np.random.default_rng(77)
    done = 0
    while done < 60:
        w = wl.medium_random(rng, int(rng.integers(0, 2)))
        if w.n_stage * w.r_max * w.c_max > 32767:
            continue
        d = rng.integers(0, 1500, size=w.coef.shape[:-1]) if rng.random() < 0.5 else None
        w = w.with_model(int(rng.integers(0, 3)), d)
        print(f"[case] stages, draw {done}", flush=True)
        same(by_stages(T, w, int(rng.integers(0, 4))), oracle.solve(w, threads=8))
        done += 1
