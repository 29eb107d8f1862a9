"""Permanents in one launch: at the edges of its workgroup and wavefront counts,
column paddings and radices, repeated, alternating and replayed from a graph."""
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
    ([1], [1]),                                     # one term
    ([0, 3], [2, 1]),                               # one row on the cheaper side
    ([1] * 7, [1] * 7), ([1] * 8, [1] * 8),         # one wavefront; the last state without time digits and the first with
    ([1] * 12, [1] * 12), ([1] * 13, [1] * 13),     # one workgroup, and two: the ticket
    ([1] * 17, [1] * 17),                           # an odd column count beyond 16 (two column registers)
    ([1] * 20, [1] * 20),
    ([2, 2, 2], [2, 2, 2]),                         # mixed radices, idle lanes
    ([3, 1, 2, 0, 2], [1, 1, 1, 4, 1]),
    ([2] * 8, [1] * 16),                            # unit powers over radix 3, the other side iterated
    ([5, 4, 3, 2], [4, 4, 3, 3]),
    ([7, 6, 5], [6, 6, 6]),
    ([1] * 4 + [2] * 4, [2] * 4 + [1] * 4),
    ([2] * 12, [2] * 12),                           # 9 * 3^6 time states on several workgroups
]


def value(eng, U, S, T):
    perm, amp = eng.perm(U, S, T)
    return complex(perm.item()), complex(amp.item())


@pytest.mark.parametrize("S,T", CASES)
def test_one_launch_matches_oracle(eng, S, T):
    m, n = len(S), sum(S)
    if len(T) != m:
        m = max(len(S), len(T))
        S, T = S + [0] * (m - len(S)), T + [0] * (m - len(T))
    U = workloads.haar(m, 500 + n + m)
    d = torch.from_numpy(U).cuda()
    got, amp = value(eng, d, S, T)
    ref = oracle.perm_mult_quad(U, np.array(S, np.int32), np.array(T, np.int32))[0]
    assert abs(got - ref) <= max((1e-10 if n <= 20 else 1e-8) * abs(ref), floor_of(U, S, T)), (got, ref)
    assert abs(amp - got * oracle.normaliser(S, T)) <= 1e-13 * abs(got)
    assert value(eng, d, S, T) == (got, amp)


def test_alternating_sizes_and_leading_dimension(eng):
    # calls of different grids share the ticket; a matrix inside a wider buffer
    U = workloads.haar(20, 1)
    wide = torch.zeros((20, 27), dtype=torch.complex128, device="cuda")
    wide[:, :20] = torch.from_numpy(U)
    sizes = [3, 13, 20, 8, 17, 20, 3, 15]
    once = {n: value(eng, torch.from_numpy(U).cuda(), [1] * n + [0] * (20 - n), [1] * n + [0] * (20 - n)) for n in set(sizes)}
    for _ in range(5):
        for n in sizes:
            assert value(eng, wide[:, :20], [1] * n + [0] * (20 - n), [1] * n + [0] * (20 - n)) == once[n]


def test_non_finite_entries(eng):
    # entries outside the pattern's rows and columns are not read; inside, they show
    U = workloads.haar(6, 3)
    S, T = [1, 1, 1, 1, 0, 0], [1, 1, 1, 0, 1, 0]
    clean = value(eng, torch.from_numpy(U).cuda(), S, T)
    V = U.copy()
    V[3, :] = np.nan
    V[:, 5] = np.inf
    assert value(eng, torch.from_numpy(V).cuda(), S, T) == clean
    V = U.copy()
    V[0, 0] = np.nan
    assert np.isnan(value(eng, torch.from_numpy(V).cuda(), S, T)[0].real)


def test_graph_replays(eng):
    # captured on a stream, replayed with other work between
    U = torch.from_numpy(workloads.haar(16, 5)).cuda()
    S = T = [1] * 15 + [0]
    want = value(eng, U, S, T)
    perm = torch.zeros((), dtype=torch.complex128, device="cuda")
    amp = torch.zeros_like(perm)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        eng.perm(U, S, T, out_perm=perm, out_amp=amp)
    other = [1] * 13 + [0] * 3
    keep = value(eng, U, other, other)
    for _ in range(4):
        perm.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert (complex(perm.item()), complex(amp.item())) == want
        assert value(eng, U, other, other) == keep
    U2 = workloads.haar(16, 6)
    U.copy_(torch.from_numpy(U2))
    g.replay()
    torch.cuda.synchronize()
    assert complex(perm.item()) == value(eng, torch.from_numpy(U2).cuda(), S, T)[0]
