"""Which step of the one-wavefront solve found each answer: it is kept with the results in
the workspace (csrc/themis_internal.h: the record per instance at the start of the table
region, KEEP_STATUS, KEEP_STEP)."""

import numpy as np

STEPS = ("A", "B", "C", "G LDS", "G HBM", "G trial", "W LDS", "W HBM", "D")


def steps_of(p, workspace):
    """step index per instance (SolveStep); -1 where there is no answer"""
    import torch
    head, per_model = 5, (6 if p.profile_form == 1 else 5) + 1 + 1 + 3
    words = head + per_model * p.n_stage
    kept = workspace[: 4 * words * p.n_inst].view(torch.int32).reshape(p.n_inst, words)
    status = kept[:, 2].cpu().numpy()
    return np.where(status & 0xFF, -1, status >> 8)
