"""Step A of the one-wavefront solve where there are more (model, batch size) pairs than lanes:
a lane takes several batch sizes of its model, from two lanes per model up to as many as leave no
gaps, or whole models take rounds (csrc/cost_front.h).  tests/host/plan_check.cpp has which shape
goes which way.  Whole numbers, so the oracle's answers word for word: no tolerance."""

import pytest

from cost_families import family
from test_gpu_cost_solve import T  # noqa: F401
from test_gpu_front import every_call

pytestmark = pytest.mark.gpu


# lanes per model and turns: 2 x 2, 4 x 4, 8 x 2; without gaps 5 x 2, 7 x 2, 6 x 3, 3 x 2;
# rounds: 2, 10 and 6; without gaps 3 and 4
@pytest.mark.parametrize("S,n_batch", [(32, 3), (16, 16), (5, 13), (11, 10), (9, 14), (10, 16), (17, 5),
                                       (64, 2), (40, 16), (22, 16), (33, 5), (23, 9)])
@pytest.mark.parametrize("queue", [0, 1, 2])
def test_lanes_and_turns(T, oracle, S, n_batch, queue):
    r_max = min(40, 32767 // (S * 7))
    w = family([S, n_batch, 8], 80, S, 7, list(range(1, n_batch + 1)), r_max, 250, S * 60_000, (10, 900))
    w = w.with_model(queue, None)
    print(f"[case] {S} models, {n_batch} batch sizes, queue {queue}", flush=True)
    want = every_call(T, oracle, w, min(r_max, 6))
    assert (want[0] == 0).any()
