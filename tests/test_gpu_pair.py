"""Long collision-free permanents by pairs of columns: at both ends of their
range, with odd and even numbers of columns and pairs, a row whose last photon
is fixed, and against exact values; pq_perm_noalloc takes the same form."""
import ctypes
from math import factorial, gamma

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def eng():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_04006_amd as pq
    return pq.Engine(0)


def value(eng, U, S, T):
    perm, amp = eng.perm(U, S, T)
    return complex(perm.item()), complex(amp.item())


@pytest.mark.parametrize("n", [22, 23, 24, 25, 26])
def test_against_oracle(eng, n):
    # 22: the last below the range; 23 to 26: 12 and 13 pairs with and without padding
    A = workloads.collision_free_block(n, 40 + n)
    U = torch.from_numpy(A).cuda()
    got, amp = value(eng, U, [1] * n, [1] * n)
    ref = oracle.perm_ryser(A)
    assert abs(got - ref) <= 1e-8 * abs(ref)
    assert amp == got
    assert value(eng, U, [1] * n, [1] * n) == (got, amp)


def low_rank_perm(n, seed):
    """A matrix whose permanent has a closed form: x_i + y_i z_j, entries of
    modulus one.  With (value, size): size bounds the rounding of a sum over
    sign vectors.  Its terms are prod_j (X + z_j Y) with X = sum +-x_i and Y
    likewise, about independent complex normals of variance n; so the mean
    modulus of a term is about E (|X|^2 + |Y|^2)^(n/2) <= 2^(n/2) n^(n/2) Gamma(n/2 + 2),
    and every term carries about n + 1 roundings."""
    rng = np.random.default_rng(seed)
    x, y, z = (np.exp(2j * np.pi * rng.random(n)) for _ in range(3))
    A = x[:, None] + y[:, None] * z[None, :]
    # sum over subsets R of rows taking the second part: prod_{R} y prod_{not R} x
    # times |R|! (n - |R|)! e_{|R|}(z)
    ez = [1.0 + 0j] + [0j] * n
    for v in z:
        for k in range(n, 0, -1):
            ez[k] = ez[k] + v * ez[k - 1]
    ey = [1.0 + 0j] + [0j] * n          # by number of rows taking y
    for a, b in zip(x, y):
        for k in range(n, 0, -1):
            ey[k] = a * ey[k] + b * ey[k - 1]
        ey[0] = a * ey[0]
    terms = [factorial(k) * factorial(n - k) * ey[k] * ez[k] for k in range(n + 1)]
    size = 16 * (n + 1) * np.finfo(float).eps * (2 * n) ** (n / 2) * gamma(n / 2 + 2)
    assert size < 1e-4 * abs(sum(terms))
    return A, sum(terms), size


@pytest.mark.parametrize("n", [25, 27, 28, 29, 30, 31, 32])
def test_closed_form(eng, n):
    # where the oracle's 2^n terms take too long
    A, want, size = low_rank_perm(n, n)
    got, _ = value(eng, torch.from_numpy(A).cuda(), [1] * n, [1] * n)
    assert abs(got - want) <= size


@pytest.mark.parametrize("n", [26, 29])
def test_wide_matrix_both_orientations_and_scale(eng, n):
    # modes picked out of a wider matrix with a leading dimension, rows and
    # columns exchanged, and the value of a scaled matrix
    A, want, size = low_rank_perm(n, 100 + n)
    rng = np.random.default_rng(n)
    m = n + 7
    rows, cols = rng.permutation(m)[:n], rng.permutation(m)[:n]
    rows.sort()
    cols.sort()
    W = np.full((m, m + 3), np.nan, dtype=np.complex128)
    W[np.ix_(rows, cols)] = A
    T = [int(i in rows) for i in range(m)]
    S = [int(j in cols) for j in range(m)]
    U = torch.from_numpy(W).cuda()[:, :m]
    got, _ = value(eng, U, S, T)
    assert abs(got - want) <= size
    Ut = torch.from_numpy(np.ascontiguousarray(W[:, :m].T)).cuda()
    swapped, _ = value(eng, Ut, T, S)
    assert abs(swapped - want) <= size
    half, _ = value(eng, U * 0.5, S, T)
    assert half == got * 0.5 ** n       # powers of two commute with every rounding


def test_row_with_two_photons(eng):
    # one doubled output mode: its last photon is the fixed one, every digit binary
    n = 26
    A, want, size = low_rank_perm(n, 7)
    A[1] = A[0]
    # perm with the repeated row by the closed form of the repeated parameters
    B = A.copy()
    U = torch.from_numpy(B).cuda()
    full, _ = value(eng, U, [1] * n, [1] * n)
    merged, _ = value(eng, U, [1] * n, [2, 0] + [1] * (n - 2))
    assert abs(full - merged) <= 2 * size


def test_non_finite_entry_shows(eng):
    n = 25
    A = workloads.collision_free_block(n, 3)
    A[4, 9] = complex(np.nan, 0.0)
    got, _ = value(eng, torch.from_numpy(A).cuda(), [1] * n, [1] * n)
    assert np.isnan(got.real) or np.isnan(got.imag)


@pytest.mark.parametrize("n", [25, 28])
def test_noalloc_same_value(eng, n):
    import paper_2403_04006_amd as pq
    lib = pq._lib.load()
    A, _, _ = low_rank_perm(n, 60 + n)
    U = torch.from_numpy(A).cuda()
    want = value(eng, U, [1] * n, [1] * n)[0]
    ones = (ctypes.c_int32 * n)(*([1] * n))
    out = torch.zeros(1, dtype=torch.complex128, device="cuda")
    st = lib.pq_perm_noalloc(eng._ctx, U.data_ptr(), n, n, ones, ones, out.data_ptr(), None,
                             torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert st == 0 and complex(out.item()) == want
