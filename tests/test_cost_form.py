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
