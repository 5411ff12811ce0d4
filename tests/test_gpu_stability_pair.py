"""The stability test with a wavefront for each of its two solves, on both sides of the batch
size up to which it has them (28 instances per compute unit), with one model and several, and
with predicted rates that are the current one, differ, or are not valid.  Whole numbers, so the
oracle's answers word for word: no tolerance."""

import numpy as np
import pytest

from cost_families import families, family
from test_gpu_cost_solve import T, same  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("more", [None, 0, 1])
@pytest.mark.parametrize("name", ["one model", "three models", "eight models", "sixteen models"])
def test_two_solves(T, oracle, name, more):
    import torch
    w = (family(16, 300, 16, 6, [1, 2, 4, 8, 16], 300, 250, 900_000, (20, 3000)) if name == "sixteen models"
         else families(300)[name])
    rng = np.random.default_rng(len(name))
    w.lam[7] = 0
    pred = np.where(rng.random(300) < 0.4, w.lam, w.lam + rng.integers(-3, 40, 300)).astype(np.int32)
    pred[11] = 0
    cores = rng.integers(1, w.c_max + 1, (300, w.n_stage)).astype(np.int32)
    n = 300 if more is None else 28 * torch.cuda.get_device_properties(0).multi_processor_count + more
    again = np.arange(n) % 300
    b = T.DeviceBatch(w.take(again))
    print(f"[case] stability {name}, {n} instances", flush=True)
    for given in (None, cores):
        want = oracle.stability(w, pred, given)
        for _ in range(2):  # what the first call leaves in LDS is no answer of the second
            stable = b.check_stability(pred[again], None if given is None else given[again])
            assert (stable.cpu().numpy() == want[0][again]).all()
            same(b.results(), tuple(x[again] for x in want[1:]))
    assert 0 < want[0].mean() < 1
