"""Which step of the one-wavefront solve found each answer: it is kept with the results in
the workspace (csrc/themis_internal.h: the record per instance at the start of the table
region, KEEP_STATUS, KEEP_STEP)."""

import numpy as np

STEPS = ("A", "B8", "B16", "C", "G LDS", "G HBM", "G trial", "W LDS", "W HBM", "D")


def steps_of(p, workspace):
    """step index per instance (SolveStep); -1 where there is no answer"""
    import torch
    head, per_model = 5, (6 if p.profile_form == 1 else 5) + 1 + 1 + 3
    words = head + per_model * p.n_stage
    kept = workspace[: 4 * words * p.n_inst].view(torch.int32).reshape(p.n_inst, words)
    status = kept[:, 2].cpu().numpy()
    return np.where(status & 0xFF, -1, status >> 8)


def steps_by_rule(w, oracle, want, cores=None):
    """The step that csrc/cost_front.h's rule (Front::reach_of) and the answers `want` make it,
    per instance; "" where there is no answer, it lies beyond the 64 cells of step C, or
    the rule's two sides are too close to call.
    cores: those of the horizontal solve."""
    lt, cost, _ = oracle.candidates(w)
    if cores is not None:
        mine = np.arange(lt.shape[-1]) // len(w.batch_sizes) + 1 == cores[..., None]
        lt = np.where(mine, lt, -1)
    cost = np.where(lt >= 0, cost, 1 << 20)
    base = cost.min(axis=2)
    ticks = np.where((lt >= 0) & (cost == base[..., None]), lt, 1 << 20).min(axis=2).sum(axis=1)
    least = np.where(lt >= 0, lt, 1 << 20).min(axis=2).sum(axis=1)
    T = w.slo_us // w.tick_us
    x = want[1] - base.sum(axis=1)
    late, gain = ticks - T, ticks - least
    given, one = w.r_fixed is not None, cores is not None or w.c_max == 1
    # the fastest candidate that the rule looks at has the most cores that make a difference
    last = np.clip(np.broadcast_to(w.coef[..., 3], base.shape), 1, w.c_max) if cores is None else cores
    at_cap = np.arange(lt.shape[-1]) // len(w.batch_sizes) + 1 == last[..., None]
    fast = np.where((lt >= 0) & at_cap, lt.astype(np.int64) << 15 | cost, 1 << 45).min(axis=2) & 0x7FFF
    late_f, gain_f = late.astype(np.float32), gain.astype(np.float32)
    have = late_f * np.sqrt(np.sqrt((fast - base).sum(axis=1).clip(0).astype(np.float32)))
    need = np.float32(1.1) * gain_f - late_f
    bounds = (2.6, np.inf) if one else (2.6, 7.0) if given else (4.5, 11.0)
    # (the square roots of the two sides may differ in the last bits)
    near = np.any([np.abs(have - b * need) <= 1e-5 * have for b in bounds if b < np.inf], axis=0)
    near |= np.abs(late_f - 0.3 * gain_f) <= 1e-5 * gain_f if not given else False
    steps = []
    for i in range(w.n_inst):
        cells = (4 if not given and late[i] <= 0.3 * gain[i] else
                 8 if have[i] <= bounds[0] * need[i] else 16 if one or have[i] <= bounds[1] * need[i] else 64)
        cells = 8 if one and cells == 4 else cells
        steps.append("" if want[0][i] != 0 or near[i] else "A" if late[i] <= 0 else
                     "B8" if x[i] < cells <= 8 else "B16" if x[i] < 16 and cells <= 16 else
                     "C" if x[i] < 64 else "")
    return np.array(steps)
