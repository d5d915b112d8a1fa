"""The slope bound of the search with weight samples (CPU): Algorithm 1's time, with both host streams
longer by the same length, never grows by less than the least slope over the orders in which the streams
may finish; over the orders that start with GPU-GPU (and compute after it) when they do so at the start."""

import itertools

import numpy as np
import pytest

from oracle import oracle as O
from paper_2503_19050_amd import workloads as W


def _slope(phi, first):
    """Least directional derivative along (0, 0, 1, 1) over the finishing orders starting with `first`."""
    least = np.inf
    for order in itertools.permutations(range(4)):
        if order[:len(first)] != first:
            continue
        x, T, mask = [0.0, 0.0, 1.0, 1.0], 0.0, 15
        for i in range(3):
            ov = x[order[i]] * phi[mask][order[i]]
            T += ov
            x = [x[j] - ov / phi[mask][j] if mask >> j & 1 else x[j] for j in range(4)]
            mask &= ~(1 << order[i])
        least = min(least, T + x[order[3]])
    return least


@pytest.mark.parametrize("hi", [1.0, 1.5, 50.0])
def test_time_grows_at_least_with_the_slope(hi):
    rng = np.random.default_rng(int(hi * 10))
    for case in range(300):
        phi = np.array(W.hw_sample(case)["phi"]) if hi == 1.5 else 1.0 + (hi - 1.0) * rng.random((16, 4))
        x = rng.choice([0.0, 1.0], 4, p=[0.1, 0.9]) * 10.0 ** rng.uniform(-2, 2, 4)
        x[0] = max(x[0], 0.01)
        first = ()
        s = x * phi[15]
        if 0.0 < s[1] < min(s[0], s[2], s[3]):
            first = (1,)
            y = (s - s[1]) / phi[15] * phi[13]
            if y[0] < min(y[2], y[3]):
                first = (1, 0)
        slope = _slope(phi, first)
        assert slope >= _slope(phi, ()) - 1e-12
        T0 = O.interference(x, phi)
        for length in 10.0 ** rng.uniform(-3, 3, 8):
            T = O.interference(x + np.array([0.0, 0.0, length, length]), phi)
            assert T >= T0 + slope * length - 1e-10 * (T0 + (1 + abs(slope)) * length)
