"""The solve that handles every distinct instance once, on a batch as it is and on its instances
again and again beyond the batch size (an instance per SIMD) up to which every instance is
solved: there they are looked for, listed, solved and handed out."""

import numpy as np

NAMES = ("status", "cost", "ticks", "cfg")


def side_by_side():
    """The most instances that are solved as they are."""
    import torch
    return 4 * torch.cuda.get_device_properties(0).multi_processor_count


def beyond(n):
    """Indices of n instances, again and again, one more than are solved as they are or more."""
    return np.arange(max(side_by_side() + 1, n)) % n


def records(b, ws):
    """The record per instance that a one-wavefront solve leaves (csrc/themis_internal.h)."""
    import torch
    words = 5 + ((6 if b.p.profile_form == 1 else 5) + 1 + 1 + 3) * b.p.n_stage
    return ws[:4 * words * b.p.n_inst].view(torch.int32).reshape(b.p.n_inst, words)


def distinct(T, w, want, prune=0, stream=None, sizes=(None, "beyond")):
    """Both batches against the pool's answers `want`, and which instances were solved."""
    import torch
    for size in sizes:
        again = np.arange(w.n_inst) if size is None else beyond(w.n_inst)
        b = T.DeviceBatch(w.take(again), prune=prune)
        b.solve_distinct()  # (and a workspace)
        ws = b.memo_workspace
        if w.n_stage <= 64:
            records(b, ws).fill_(0x11111111)
        for out in (b.status, b.cost, b.ticks, b.cfg):
            out.fill_(77)
        torch.cuda.synchronize()
        b.solve_distinct(stream=stream)
        torch.cuda.synchronize()
        for name, g, x in zip(NAMES, b.results(), want):
            bad = np.nonzero((g != x[again]).reshape(len(again), -1).any(axis=1))[0]
            assert bad.size == 0, f"{len(again)} instances: {name} differs at {bad[:8]}"
        if w.n_stage <= 64:
            solved = int((records(b, ws)[:, 2] != 0x11111111).sum())
            if len(again) <= side_by_side():
                assert solved == len(again)
            else:
                tuples = [w.lam[:, None], w.slo_us[:, None]]
                if not w.coef_shared:
                    tuples.append(w.coef.reshape(w.n_inst, -1))
                if w.r_fixed is not None:
                    tuples.append(w.r_fixed)
                different = len(np.unique(np.concatenate(tuples, axis=1), axis=0))
                assert solved == different, f"{solved} solved of {different} different instances"
