"""Gradients over the routes of the derivative reduction: a pattern's own
workgroup, one stage, two stages, and all of them in one call."""
import numpy as np
import pytest

import workloads
from tests.test_gpu_grad import check, eng  # noqa: F401

pytestmark = pytest.mark.gpu


def one_each(m, n, shift):
    v = np.zeros(m, dtype=np.int32)
    v[(np.arange(n) + shift) % m] = 1
    return v


@pytest.mark.parametrize("n", [2, 9, 10, 11, 12, 13, 14, 15, 16, 18, 20])
def test_single_pattern(eng, n):  # noqa: F811
    # one pattern alone is cut into the most chunks
    m = n + 2
    check(eng, workloads.haar(m, 300 + n), [one_each(m, n, 0)], [one_each(m, n, 1)], [0.5 - 1.25j])


@pytest.mark.parametrize("shape", [(4, 4, 3), (5, 5, 4, 2), (2, 2, 2, 2, 2, 2, 2)])
def test_single_pattern_with_repeats(eng, shape):  # noqa: F811
    S = np.array(shape, dtype=np.int32)
    check(eng, workloads.haar(len(S), 320 + len(S)), [S], [S[::-1].copy()], [1.0 + 0.25j])


def test_all_routes_in_one_call(eng):  # noqa: F811
    m = 19
    ns = [18, 3, 13, 15, 3, 18, 1, 16]
    Ss = [one_each(m, n, k) for k, n in enumerate(ns)]
    Ts = [one_each(m, n, 2 * k + 1) for k, n in enumerate(ns)]
    Ss[4], Ts[4] = Ss[1], Ts[1]      # a copy
    Ss[6] = np.zeros(m, dtype=np.int32)
    Ts[6] = np.zeros(m, dtype=np.int32)      # no photons
    g = [complex(1 + k, 0.5 * k) for k in range(len(ns))]
    check(eng, workloads.haar(m, 333), Ss, Ts, g)
