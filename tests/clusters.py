"""Compact clusters that put all centres into one neighbour count (test helper)."""

import numpy as np


def compact_cluster(atoms, seed):
    """The grid points nearest to a grid's centre, 0.95 A apart with a little jitter: every pair
    of up to 121 atoms is within the cutoff."""
    rng = np.random.default_rng(seed)
    g = np.stack(np.meshgrid(*[np.arange(-4, 5) * 0.95] * 3, indexing="ij"), -1).reshape(-1, 3)
    x = g[np.argsort((g * g).sum(1), kind="stable")[:atoms]]
    return x + rng.uniform(-0.03, 0.03, x.shape), rng.integers(0, 5, atoms).astype(np.int32)
