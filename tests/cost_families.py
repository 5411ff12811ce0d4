"""Batches whose answers cost far more than the least the models can be run with:
the recurrence over the cost (csrc/cost_solve.hip) is then as long as it gets."""

import numpy as np

from paper_2407_14843_amd import workloads as wl


def family(seed, n, n_stage, c_max, batch_sizes, r_max, tick, slo_max, lam, r_fixed=0):
    rng = np.random.default_rng(seed)
    coef = wl._draw_coef(rng, (n, n_stage), a=(1000, 40000), k=(100, 10000), q=(0, 100),
                         p=(1, c_max), o=(1, 2000))
    rate = np.rint(np.exp(rng.uniform(np.log(lam[0]), np.log(lam[1]), n))).astype(np.int32)
    slo = rng.integers(0, slo_max + 1, n).astype(np.int32)
    given = rng.integers(1, r_fixed + 1, (n, n_stage)).astype(np.int32) if r_fixed else None
    return wl.Workload("cost", wl.VERTICAL if r_fixed else wl.JOINT, n, n_stage, c_max,
                       batch_sizes, r_max, tick, slo_max, False, coef, rate, slo, r_fixed=given)


def families(n):
    """name -> workload of n instances"""
    return {
        # one core per replica, thousands of replicas: costs spread over thousands
        "three models": family(1, n, 3, 1, [1, 2, 4, 8, 16, 32, 64], 10000, 500, 400_000,
                               (1000, 200_000)),
        "four models": family(2, n, 4, 1, [1, 3, 9, 27, 81], 8000, 250, 500_000,
                              (100_000, 1_000_000)),
        # more than 64 (model, batch size) pairs
        "eight models": family(4, n, 8, 2, [1, 2, 3, 4, 5, 6, 7, 8, 16], 2000, 250, 700_000,
                               (10, 100_000)),
        "ten models, replicas given": family(5, n, 10, 16, [1, 2, 4, 8], 8, 1000, 1_000_000,
                                             (10, 2000), r_fixed=8),
        # more core counts than the table of reciprocals holds
        "many cores": family(6, n, 2, 150, [1, 2, 5], 100, 500, 100_000, (10, 20_000)),
        # lists of candidates longer than a compute unit full of wavefronts has room for,
        # and costs spread over thousands
        "long lists": family(11, n, 3, 64, list(range(1, 17)), 150, 50, 40_000,
                             (20_000, 400_000)),
        "one model": family(7, n, 1, 6, [1, 2, 4], 50, 100, 60_000, (1, 3000)),
    }


def over_base(w, oracle, solved):
    """Cost of every solved instance above the least its models can be run with."""
    lt, cost, _ = oracle.candidates(w)
    base = np.where(lt >= 0, cost, 1 << 20).min(axis=2).sum(axis=1)
    return (solved[1] - base)[solved[0] == 0]
