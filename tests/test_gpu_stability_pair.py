"""The stability test with a wavefront for each of its two solves, on both sides of the batch
size up to which it has them (28 instances per compute unit), with one model and several, and
with predicted rates that are the current one, differ, or are not valid.  Whole numbers, so the
oracle's answers word for word: no tolerance."""

import numpy as np
import pytest

from cost_families import families, family
from solve_steps import STEPS, steps_of
from test_gpu_cost_solve import T, same  # noqa: F401

pytestmark = pytest.mark.gpu


def in_pairs():
    """The most instances that have two wavefronts each."""
    import torch
    return 28 * torch.cuda.get_device_properties(0).multi_processor_count


# (beyond the bound the queue models: each has a kernel of its own)
@pytest.mark.parametrize("more,queue", [(None, 0), (0, 0), (1, 0), (None, 1), (None, 2), (1, 1), (1, 2)])
@pytest.mark.parametrize("name", ["one model", "three models", "eight models", "sixteen models"])
def test_two_solves(T, oracle, name, more, queue):
    w = (family(16, 300, 16, 6, [1, 2, 4, 8, 16], 300, 250, 900_000, (20, 3000)) if name == "sixteen models"
         else families(300)[name]).with_model(queue, None)
    rng = np.random.default_rng(len(name))
    w.lam[7] = 0
    pred = np.where(rng.random(300) < 0.4, w.lam, w.lam + rng.integers(-3, 40, 300)).astype(np.int32)
    pred[11] = 0
    cores = rng.integers(1, w.c_max + 1, (300, w.n_stage)).astype(np.int32)
    n = 300 if more is None else in_pairs() + more
    again = np.arange(n) % 300
    b = T.DeviceBatch(w.take(again))
    print(f"[case] stability {name}, {n} instances, queue {queue}", flush=True)
    for given in (None, cores):
        want = oracle.stability(w, pred, given)
        for _ in range(2):  # what the first call leaves in LDS is no answer of the second
            stable = b.check_stability(pred[again], None if given is None else given[again])
            assert (stable.cpu().numpy() == want[0][again]).all()
            same(b.results(), tuple(x[again] for x in want[1:]))
    assert 0 < want[0].mean() < 1


# Lanes per model 4, 8 and 16, pairs without gaps, in turns and in rounds of models: beyond the
# bound, where an instance's solves share a wavefront.
@pytest.mark.parametrize("S,n_batch", [(16, 4), (8, 7), (4, 16), (7, 9), (9, 9), (33, 2)])
def test_one_wavefront(T, oracle, S, n_batch):
    w = family([S, n_batch], 240, S, 7, list(range(1, n_batch + 1)), min(40, 32767 // (S * 7)), 250,
               S * 60_000, (10, 900))
    pred = np.maximum(1, w.lam + np.random.default_rng(S).integers(-3, 4, 240)).astype(np.int32)
    want = oracle.stability(w, pred)
    again = np.arange(in_pairs() + 1) % 240
    print(f"[case] stability {S} models, {n_batch} batch sizes, {again.size} instances", flush=True)
    b = T.DeviceBatch(w.take(again))
    stable = b.check_stability(pred[again])
    assert (stable.cpu().numpy() == want[0][again]).all()
    same(b.results(), tuple(x[again] for x in want[1:]))
    assert 0 < want[0].mean() < 1


# An instance's rows by cost in HBM are one region, which the second wavefront waits for.  Which
# instances use it is what the horizontal solve at either rate says, of a batch whose
# wavefronts have as much LDS or more.
@pytest.mark.parametrize("S,n,lam,slo,given", [(64, 1000, (10, 2000), 4_000_000, False),
                                               (64, 700, (500, 20_000), 4_000_000, True),
                                               (32, 1500, (10, 2000), 2_000_000, True)])
def test_rows_in_hbm_of_both(T, oracle, S, n, lam, slo, given):
    w = family(3, 96, S, 8, [1, 2, 4, 8], 32767 // (S * 8) // 2, 500, slo, lam)
    rng = np.random.default_rng(S)
    pred = (w.lam + rng.integers(1, 3, 96)).astype(np.int32)
    cores = np.random.default_rng(5).integers(1, 9, (96, S)).astype(np.int32) if given else None

    def in_hbm(rates):
        v = w.take(np.arange(2 * n) % 96)
        v.lam = rates[np.arange(2 * n) % 96]
        b = T.DeviceBatch(v)
        b.solve_horizontal(cores if cores is None else cores[np.arange(2 * n) % 96])
        step = steps_of(b.p, b.workspace)[:96]
        return np.isin(step, [STEPS.index(s) for s in ("G HBM", "W HBM", "D")])

    at = np.nonzero(in_hbm(w.lam) & in_hbm(pred))[0]
    print(f"[case] stability {S} models, {at.size} instances with both rows in HBM", flush=True)
    assert at.size >= 2
    want = oracle.stability(w, pred, cores)
    # as a batch of all instances, and of those only
    for pick in (np.arange(n) % 96, at[np.arange(n) % at.size]):
        b = T.DeviceBatch(w.take(pick))
        for _ in range(3):
            stable = b.check_stability(pred[pick], cores if cores is None else cores[pick])
            assert (stable.cpu().numpy() == want[0][pick]).all()
            same(b.results(), tuple(x[pick] for x in want[1:]))


# A current rate beyond what the most replicas can take: nothing is stable, and the solve at the
# predicted rate ends before the long steps (its results lie behind the workspace of one solve).
@pytest.mark.parametrize("S,n_batch,queue", [(3, 7, 0), (8, 7, 0), (16, 4, 0), (16, 7, 1), (9, 9, 2),
                                             (33, 2, 0), (64, 4, 0)])
@pytest.mark.parametrize("share", [1.0, 0.5])
def test_a_second_solve_in_vain(T, oracle, S, n_batch, queue, share):
    w = family([S, 5], 240, S, 8, [2 ** j for j in range(n_batch)], 32767 // (S * 8) // 2, 500,
               min(S * 60_000, 4_000_000), (500, 20_000) if S < 33 else (10, 2000)).with_model(queue, None)
    pred = w.lam.copy()
    now = w.take(np.arange(240))
    beyond = np.random.default_rng(S).random(240) < share
    now.lam = np.where(beyond, 1 << 20, np.maximum(1, w.lam - 1)).astype(np.int32)
    want = oracle.stability(now, pred)
    h = T.DeviceBatch(w)
    h.solve_horizontal(None)
    long = np.array([s.startswith("G") for s in STEPS + ("",)])[steps_of(h.p, h.workspace)]
    none = long & (want[1] == T.INFEASIBLE)
    print(f"[case] stability {S} models, {none.sum()} long solves in vain", flush=True)
    assert none.any()
    b = T.DeviceBatch(now)
    for _ in range(2):
        stable = b.check_stability(pred).cpu().numpy()
        assert (stable == want[0]).all()
        same(b.results(), want[1:])
        behind = b.stability_workspace[T.workspace_bytes(b.p):][:4 * 240].cpu().numpy().view(np.int32)
        assert not (behind[none] == T.SOLVED).any()
        assert (behind[long & (want[1] == T.SOLVED)] == T.SOLVED).all()
