"""Step C of the one-wavefront solve (csrc/cost_solver.h, solve_sixtyfour): the recurrence over
64 cells at the fewest models and at more than a wavefront's rows of 32 words, with candidates
of both parities and halves of the table, and answers up to the last cell.  Whole numbers, so
the oracle's answers word for word: no tolerance."""

import numpy as np
import pytest

from cost_families import family, over_base
from solve_steps import STEPS, steps_of
from test_gpu_cost_solve import T, same  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,r_max,lam", [(2, 60, (2000, 20_000)), (3, 60, (2000, 20_000)),
                                         (9, 60, (200, 4000)), (16, 30, (50, 1500)),
                                         (33, 20, (30, 500)), (64, 20, (20, 200))])
def test_every_cell(T, oracle, S, r_max, lam):
    w = family([S, 64], 3000 if S < 33 else 800, S, 16 if S < 33 else 8, [1, 2, 4, 8, 16], r_max, 250,
               S * 60_000, lam)
    want = oracle.solve(w, threads=8)
    over = over_base(w, oracle, want)
    at = np.nonzero(want[0] == 0)[0][over < 64]
    w, want, over = w.take(at), tuple(x[at] for x in want), over[over < 64]
    print(f"[case] step C, {S} models, {len(at)} instances", flush=True)
    b = T.DeviceBatch(w)
    b.solve()
    same(b.results(), want)
    by_c = np.array(STEPS)[steps_of(b.p, b.workspace)] == "C"
    # answers below and from 32 cells on, even and odd
    met = {(x >= 32, x % 2) for x in over[by_c].tolist()}
    assert len(met) == 4, (met, by_c.sum())
