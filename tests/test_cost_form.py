"""The recurrence over the total cost gives the answers of the one over the budget:
a plain implementation of it on the CPU checker's candidate tables against the
checker's own solve, on batches whose answers lie anywhere from 0 to thousands of
cores above the least."""

import numpy as np
import pytest

from cost_families import families


def solve_by_cost(lt, cost, T):
    """One instance; lt, cost [S][K], lt = -1 where infeasible."""
    S = len(lt)
    feas = [np.nonzero(lt[s] >= 0)[0] for s in range(S)]
    if any(f.size == 0 for f in feas) or sum(lt[s][f].min() for s, f in enumerate(feas)) > T:
        return None
    base = [cost[s][f].min() for s, f in enumerate(feas)]
    width = 64
    while True:
        rows = [np.zeros(width, np.int64)]
        for s in range(S - 1, -1, -1):
            row = np.full(width, 1 << 30)
            for k in feas[s]:
                d = cost[s][k] - base[s]
                if d < width:
                    row[d:] = np.minimum(row[d:], rows[-1][:width - d] + lt[s][k])
            rows.append(row)
        rows.reverse()
        if rows[0][-1] <= T:
            break
        width *= 4
    x = total = int(np.argmax(rows[0] <= T))
    t = ticks = int(rows[0][x])
    ks = []
    for s in range(S):
        for k in feas[s]:  # ascending: the first that continues the optimum
            d = int(cost[s][k] - base[s])
            if d <= x and lt[s][k] + rows[s + 1][x - d] == t:
                break
        else:
            raise AssertionError("no candidate continues the optimum")
        ks.append(int(k))
        x, t = x - d, t - int(lt[s][k])
    return total + int(sum(base)), ticks, ks


@pytest.mark.parametrize("name", list(families(1)))
def test_cost_recurrence_gives_the_same_answers(oracle, name):
    w = families(60)[name]
    status, cost, ticks, cfg = oracle.solve(w, threads=8)
    lt, co, rep = oracle.candidates(w)
    nb = len(w.batch_sizes)
    for i in range(w.n_inst):
        got = solve_by_cost(lt[i], co[i], int(w.slo_us[i]) // w.tick_us)
        assert (got is None) == (status[i] == 1)
        if got is None:
            continue
        want = [(k // nb + 1, w.batch_sizes[k % nb], rep[i, s, k]) for s, k in enumerate(got[2])]
        assert got[:2] == (cost[i], ticks[i]) and (np.array(want) == cfg[i]).all(), i


def within_the_gap(lt, cost, T):
    """Per model the candidates that Lagrangian bounds leave (step G's argument, in double
    precision): the hull walk between the cheapest and the fastest assignment, the cost `ub`
    of the faster end after one change of a choice, and cost + mu lt at most ub - bound over
    the model's least."""
    S = range(len(lt))
    total = lambda w: (sum(int(cost[s][w[s]]) for s in S), sum(int(lt[s][w[s]]) for s in S))
    cheap = [np.lexsort((lt[s], cost[s]))[0] for s in S]
    fast = [np.lexsort((cost[s], lt[s]))[0] for s in S]
    (c0, l0), (c1, l1) = total(cheap), total(fast)
    assert l1 <= T < l0
    while True:
        mu = (c1 - c0) / (l0 - l1)
        y = [cost[s] + mu * lt[s] for s in S]
        w = [int(np.argmin(v)) for v in y]
        c, t = total(w)
        if c * (l0 - l1) + (c1 - c0) * t >= c1 * (l0 - l1) + (c1 - c0) * l1:
            break
        if t <= T:
            c1, l1, fast = c, t, w
        else:
            c0, l0 = c, t
        if c0 >= c1:
            break
    ub = c1
    for s in S:
        fits = lt[s] - lt[s][fast[s]] <= T - l1
        ub = min(ub, c1 + int((cost[s] - cost[s][fast[s]])[fits].min()))
    gap = ub - (sum(v.min() for v in y) - mu * T)
    assert gap >= -1e-6 * ub
    return ub, [v - v.min() <= gap + 1e-6 * ub for v in y]


@pytest.mark.parametrize("name", [n for n in families(1) if n != "one model"])
def test_every_answer_is_within_the_gap(oracle, name):
    """No candidate of an answer is dropped, and few others are kept."""
    w = families(60)[name]
    status, cost, ticks, cfg = oracle.solve(w, threads=8)
    lt, co, _ = oracle.candidates(w)
    nb = len(w.batch_sizes)
    left = met = 0
    for i in np.nonzero(status == 0)[0]:
        feas = [np.nonzero(lt[i, s] >= 0)[0] for s in range(w.n_stage)]
        l = [lt[i, s][f].astype(np.int64) for s, f in enumerate(feas)]
        c = [co[i, s][f].astype(np.int64) for s, f in enumerate(feas)]
        cheapest = sum(int(l[s][np.lexsort((l[s], c[s]))[0]]) for s in range(w.n_stage))
        T = int(w.slo_us[i]) // w.tick_us
        if cheapest <= T:
            continue
        ub, kept = within_the_gap(l, c, T)
        assert ub >= cost[i]
        for s, f in enumerate(feas):
            k = (cfg[i, s, 0] - 1) * nb + w.batch_sizes.index(cfg[i, s, 1])
            assert kept[s][list(f).index(k)], (i, s)
        left += sum(int(k.sum()) for k in kept)
        met += sum(len(f) for f in feas)
    assert met and left < met
