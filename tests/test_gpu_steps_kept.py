"""The step that found an answer is kept with it, and stays out of the status that the
backtrack call hands out."""

import numpy as np
import pytest

from cost_families import families
from solve_steps import STEPS, steps_of
from test_gpu_cost_solve import T, backtrack, same  # noqa: F401

pytestmark = pytest.mark.gpu


def test_step_and_status(T, oracle):
    w = families(240)["eight models"]
    want = oracle.solve(w, threads=8)
    b = T.DeviceBatch(w)
    b.solve()
    same(b.results(), want)
    same(backtrack(T, b), want)
    step = steps_of(b.p, b.workspace)
    assert ((step >= 0) == (want[0] == 0)).all()
    met = {STEPS[k][0] for k in np.unique(step[step >= 0])}
    assert {"A", "B", "C", "G"} <= met, met
