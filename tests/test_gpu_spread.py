"""Short sweeps, spread over one round of wavefronts in shares of a few states,
and the step tables of mixed radices: values at the edges of the shares."""
import numpy as np
import pytest

import oracle
import workloads
from tests.tolerance import floor_of

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def eng():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_04006_amd as pq
    return pq.Engine(0)


@pytest.mark.parametrize("S,T", [
    ([1] * 10, [1] * 10),                            # 8 time states: one share
    ([1] * 11, [1] * 11),                            # 16: two
    ([1] * 19, [1] * 19),                            # 4096
    ([2] * 7, [2] * 7),                              # 27 time states, radix 3
    ([3, 3, 2, 2, 2, 2], [3, 2, 3, 2, 2, 2]),        # mixed radices
    ([6, 5, 4, 3, 2, 1], [5, 6, 3, 4, 2, 1]),        # radices 3 to 7 (every division path)
    ([4] * 8, [4] * 8),                              # radix 5: 4 * 5^7 terms
    ([9, 8, 7], [8, 8, 8]),                          # the general division
    ([2] * 13, [2] * 13),                            # 22 photons and more: several inner blocks
])
def test_short_sweeps_match_oracle(eng, S, T):
    m, n = len(S), sum(S)
    U = workloads.haar(m, 900 + n)
    perm, amp = eng.perm(torch.from_numpy(U).cuda(), S, T)
    ref = oracle.perm_mult_quad(U, np.array(S, np.int32), np.array(T, np.int32))[0]
    got = complex(perm.item())
    tol = max((1e-10 if n <= 20 else 1e-8) * abs(ref), floor_of(U, S, T))
    assert abs(got - ref) <= tol, (got, ref)
    norm = oracle.normaliser(S, T)
    assert abs(complex(amp.item()) - got * norm) <= 1e-13 * abs(got) * norm


@pytest.mark.parametrize("loops", [False, True])
@pytest.mark.parametrize("reps", [
    [2] * 7,                          # 9 time states
    [2] * 9,                          # 81
    [1] * 12,                         # unit vertices
    [3, 3, 2, 2, 2, 1, 1],            # mixed radices
    [4, 4, 4, 4, 2],                  # radix 5 lanes
])
def test_short_hafnians_match_oracle(eng, reps, loops):
    d, N = len(reps), sum(reps)
    A = workloads.gbs_matrix(d, 60 + d)
    gamma = workloads.loop_vector(d, d) if loops else None
    got = complex(eng.lhaf(torch.from_numpy(A).cuda(), None if gamma is None else torch.from_numpy(gamma).cuda(), reps).item())
    ref = oracle.lhaf_rep(A, gamma, reps)
    assert abs(got - ref) <= (1e-10 if N <= 20 else 1e-8) * abs(ref), (got, ref)
