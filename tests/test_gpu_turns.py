"""Step A of the one-wavefront solve where there are more (model, batch size) pairs than lanes:
a lane takes several batch sizes of its model (csrc/cost_front.h), with one lane per model up to
as many as leave no gaps, in two turns up to sixteen.  Whole numbers, so the oracle's answers word
for word: no tolerance."""

import pytest

from cost_families import family
from test_gpu_cost_solve import T  # noqa: F401
from test_gpu_front import every_call

pytestmark = pytest.mark.gpu


# lanes per model and turns: 1 x 2, 1 x 16, 2 x 2, 2 x 8, 4 x 4; without gaps 5 x 2, 7 x 2, 12 x 2, 6 x 3
@pytest.mark.parametrize("S,n_batch", [(64, 2), (40, 16), (32, 3), (22, 16), (16, 16),
                                       (11, 10), (9, 14), (5, 13), (10, 16)])
@pytest.mark.parametrize("queue", [0, 1, 2])
def test_lanes_and_turns(T, oracle, S, n_batch, queue):
    r_max = min(40, 32767 // (S * 7))
    w = family([S, n_batch, 8], 80, S, 7, list(range(1, n_batch + 1)), r_max, 250, S * 60_000, (10, 900))
    w = w.with_model(queue, None)
    print(f"[case] {S} models, {n_batch} batch sizes, queue {queue}", flush=True)
    want = every_call(T, oracle, w, min(r_max, 6))
    assert (want[0] == 0).any()
