"""Batches of small planes that the launch of several steps takes with 512 and with 1,024 lanes, shared by the test
of the plan and the test of its results (not a test module)."""
import numpy as np

# storage, planes, shortest and longest side, order; lanes and most steps of a launch
CASES = [("f32", 8, 10, 30, 3, 512, 8), ("f32", 8, 10, 30, 2, 512, 8), ("f64", 8, 10, 30, 3, 512, 8),
         ("f64", 8, 10, 30, 2, 512, 8), ("f32", 40, 10, 22, 2, 512, 16), ("f64", 40, 10, 22, 3, 512, 16),
         ("f64", 40, 10, 22, 2, 512, 16), ("f32", 60, 14, 32, 3, 1024, 16), ("f64", 90, 20, 44, 2, 1024, 6),
         ("f64", 90, 20, 44, 3, 1024, 6)]


def planes(count, lo, hi):
    rng = np.random.default_rng(41)
    return [tuple(int(v) for v in rng.integers(lo, hi + 1, 2)) + (1,) for _ in range(count)]
