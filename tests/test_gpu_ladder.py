"""All outputs built photon by photon (the default form of pq_perm_all_outputs)
against the oracle, at the edges of its level sizes and photon groups."""
from fractions import Fraction
from math import factorial

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EPS = float(np.finfo(np.float64).eps)


@pytest.fixture(scope="module")
def eng():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_04006_amd as pq
    return pq.Engine(0)


def two_modes_exact(U, S, T):
    """perm(U_{T,S}) on two modes in rational arithmetic: T! times the
    coefficient of x^T_0 y^T_1 in prod_j (U_0j x + U_1j y)^S_j.  (At 48 photons
    the signed sums cancel 14 digits more than the oracle's quad precision
    holds.)"""
    poly = [(Fraction(1), Fraction(0))]                     # by the power of x
    for j in range(2):
        a, b = ((Fraction(U[i, j].real), Fraction(U[i, j].imag)) for i in range(2))
        for _ in range(S[j]):
            nxt = [(Fraction(0), Fraction(0))] * (len(poly) + 1)
            for p, (re, im) in enumerate(poly):
                for q, (c, d) in ((p + 1, a), (p, b)):
                    nxt[q] = (nxt[q][0] + re * c - im * d, nxt[q][1] + re * d + im * c)
            poly = nxt
    f = factorial(int(T[0])) * factorial(int(T[1]))
    return complex(float(poly[T[0]][0] * f), float(poly[T[0]][1] * f))


@pytest.mark.parametrize("S", [
    [5],                                   # one mode, one output
    [0, 1],                                # one photon
    [1, 0, 1],                             # two photons
    [1, 2, 0, 0],                          # three: the last level without one below
    [0, 1, 1, 0, 1, 1],                    # four: one group of loads
    [3, 0, 2],                             # five: a group of one
    [1] * 8 + [0] * 3,                     # eight: two whole groups
    [9, 0, 0],                             # one input mode
    [1, 1, 1, 1, 1] + [0] * 7,             # level 5 of 12 modes is one over the small kernel's last level
    [1, 0, 1] + [0] * 61,                  # 64 modes, 2080 outputs
    [1, 1, 1] + [0] * 30,                  # 33 modes (the table's rows are padded to 64)
    [2, 2, 2, 2],                          # 8 photons in 4 modes, repeated inputs
    [24, 24],                              # the most photons
])
def test_ladder_matches_oracle(eng, S):
    # every level adds at most k + 3 roundings to a sum of products whose
    # moduli add up to the permanent of the moduli: n (n + 7) eps of it in all
    import paper_2403_04006_amd as pq
    m, n = len(S), sum(S)
    U = workloads.haar(m, 400 + m + n)
    perm, amp = eng.perm_all_outputs(torch.from_numpy(U).cuda(), S)
    only, none = eng.perm_all_outputs(torch.from_numpy(U).cuda(), S, with_amp=False)
    assert none is None and torch.equal(only, perm)
    perm, amp = perm.cpu().numpy(), amp.cpu().numpy()
    count = pq.fock_count(m, n)
    assert perm.shape == amp.shape == (count,)
    assert abs(np.sum(np.abs(amp) ** 2) - 1.0) <= 4 * n * (n + 7) * EPS * np.sqrt(count)
    rng = np.random.default_rng(count)
    ranks = {0, count - 1, *rng.integers(0, count, 40).tolist()}
    for r in ranks:
        T = np.array(pq.fock_unrank(m, n, r), np.int32)
        exact = (lambda A: two_modes_exact(A, S, T)) if n > 20 else (lambda A: oracle.perm_mult(A, S, T))
        size = abs(exact(np.abs(U).astype(complex)))
        assert abs(perm[r] - exact(U)) <= n * (n + 7) * EPS * size, (r, T)
        # exp(-lg / 2) carries the rounding of lg on both sides
        norm = oracle.normaliser(np.array(S, np.int32), T)
        lg = -2.0 * np.log(norm)
        assert abs(amp[r] - perm[r] * norm) <= (2 * n + 4 + 2 * lg) * EPS * abs(perm[r]) * norm, (r, T)
