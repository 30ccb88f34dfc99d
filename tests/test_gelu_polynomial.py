"""The scoring network's activation polynomial, read from its source: its error
against the exact GELU over a fine grid, in exact arithmetic and with every
step rounded to FP32, stays within the bounds stated beside it."""
import os
import re

import numpy as np
from scipy.special import ndtr

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2303_02650_amd", "csrc",
                   "pecc_lp.hip")


def coefficients():
    body = open(SRC).read().split("float gelu_fast(float t)")[1].split("return")[0]
    c = re.findall(r"(-?\d\.\d+e[+-]\d+)f", body)
    assert len(c) == 7
    return np.array([np.float32(v) for v in c])


def test_bounds():
    c, t = coefficients(), np.linspace(0.0, 8.0, 1000001)
    q = np.full_like(t, c[0])
    for k in c[1:]:
        q = q * t + np.float64(k)
    assert np.abs(t * np.exp2(q) - t * ndtr(-t)).max() <= 5.5e-8
    t = t.astype(np.float32).astype(np.float64)
    q = np.full_like(t, c[0])
    for k in c[1:]:
        q = (q * t + np.float64(k)).astype(np.float32).astype(np.float64)
    e = np.exp2(q).astype(np.float32).astype(np.float64)
    for x in (t, -t):
        g = (np.maximum(x, 0.0) - t * e).astype(np.float32).astype(np.float64)
        want = x * ndtr(x)
        # half a unit of the rounded sum at most on top
        assert (np.abs(g - want) - np.spacing(np.abs(want).astype(np.float32)) / 2).max() <= 8.9e-8
