"""Mixed-radix permanents over several segments and high digits: small and large
radices, one and many lane digits, general powers, short and long shares."""
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


CASES = [
    ([2] * 12, [2] * 12),                       # the last mixed one of one launch
    ([2] * 13, [2] * 13),                       # 19,683 states, high digits of radix 3
    ([1, 2] * 8, [2, 1] * 8),                   # radices 2 and 3 mixed, powers 1 and 2
    ([3] * 9, [4, 2] * 4 + [3]),
    ([4, 4, 3, 3, 4, 4, 4], [4, 4, 4, 4, 3, 3, 4]),
    ([20, 18], [19, 19]),                       # two rows: one digit is the lanes'
    ([6, 7, 5, 6, 6], [10, 10, 10, 0, 0]),      # powers beyond the grouped product's
    ([9, 2, 9, 2, 2, 2], [5, 4, 5, 4, 4, 4]),   # large and small radices
]


@pytest.mark.parametrize("S,T", CASES)
def test_matches_oracle(eng, S, T):
    m, n = len(S), sum(S)
    U = workloads.haar(m, 700 + n + m)
    perm, amp = eng.perm(torch.from_numpy(U).cuda(), S, T)
    got = complex(perm.item())
    ref = oracle.perm_mult_quad(U, np.array(S, np.int32), np.array(T, np.int32))[0]
    assert abs(got - ref) <= max((1e-10 if n <= 20 else 1e-8) * abs(ref), floor_of(U, S, T)), (got, ref)
    again, _ = eng.perm(torch.from_numpy(U).cuda(), S, T)
    assert complex(again.item()) == got
