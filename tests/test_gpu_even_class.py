"""Lists with long forward jobs of 13 to 22 columns (padded to an even number)
beside short ones, on the work queue and off it, against the single sweep."""
import numpy as np
import pytest

import oracle
import workloads
from tests.test_gpu_batched import dev, eng, perm_job  # noqa: F401
from tests.tolerance import floor_of

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("queue", ["always", "never"])
@pytest.mark.parametrize("m,mult", [(13, 3), (14, 3), (16, 2), (17, 2), (18, 2), (21, 2)])
def test_long_jobs_beside_short_ones(eng, m, mult, queue):  # noqa: F811
    # the first pattern has 2^18 time states or more
    U = workloads.haar(m, 900 + m)
    pats = []
    S, T = np.full(m, mult, np.int32), np.full(m, mult, np.int32)
    S[0] -= 1
    T[m - 1] -= 1
    pats.append((S, T))
    for n in (m, m - 1, 5):
        one = np.zeros(m, np.int32)
        one[:n] = 1
        pats.append((one, one[::-1].copy()))
    eng.queue_mode(queue)
    try:
        perm, _ = eng.perm_batched(dev(U), [perm_job(S, T) for S, T in pats])
    finally:
        eng.queue_mode("auto")
    for k, (S, T) in enumerate(pats):
        got = complex(perm[k].item())
        single = complex(eng.perm(dev(U), list(S), list(T))[0].item())
        # two sums of the same terms in different orders
        assert abs(got - single) <= max(2e-10 * abs(single), 2 * floor_of(U, S, T)), (k, got, single)
        if int(S.sum()) <= 18:
            ref = complex(oracle.perm_mult(U, S, T))
            assert abs(got - ref) <= max(1e-10 * abs(ref), floor_of(U, S, T))
