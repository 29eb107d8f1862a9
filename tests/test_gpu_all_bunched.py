"""Every output of inputs that hold four or more photons in one mode: the levels
of those photons are one step, in the kernel of the small levels, in a level of
its own or in the last one."""
import functools
import math

import numpy as np
import pytest

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


def permanent(U, cols, T):
    """perm(U_{T, cols}) by expanding along the last column, 80-bit."""
    @functools.lru_cache(None)
    def value(T):
        k = sum(T)
        if k == 0:
            return np.clongdouble(1.0)
        v = np.clongdouble(0.0)
        for i, t in enumerate(T):
            if t:
                v += t * np.clongdouble(U[i, cols[k - 1]]) * value(T[:i] + (t - 1,) + T[i + 1:])
        return v
    return value(tuple(int(t) for t in T))


@pytest.mark.parametrize("S", [
    [4], [3, 0], [4, 0], [0, 4], [0, 48], [47, 1], [24, 0, 24],   # one to three modes, all in the small kernel
    [5, 0, 0, 4], [4, 4, 4], [0, 1, 9, 0, 2],
    [16, 0, 0, 0, 0, 0], [0, 13, 1, 0, 0, 0],          # the first level is the small kernel's last, and the outputs
    [0, 0, 0, 0, 10, 0, 0, 0], [2, 0, 9, 0, 0, 0, 0, 0],   # ... is a level of its own, the last and not
    [0] * 15 + [6], [1, 0, 0, 0, 0, 6] + [0] * 10, [0] * 9 + [4] + [0] * 30,
])
def test_bunched_inputs(eng, S):
    # an output adds and multiplies at most 4 n times into each of the products whose moduli add up to the permanent of
    # the moduli
    m, n = len(S), sum(S)
    U = workloads.haar(m, 30 + n)
    perm, amp = (x.cpu().numpy() for x in eng.perm_all_outputs(torch.from_numpy(U).cuda(), S))
    eng.all_outputs_gemm("never")
    sweep = eng.perm_all_outputs(torch.from_numpy(U).cuda(), S)[0].cpu().numpy()
    eng.all_outputs_gemm("auto")
    count = math.comb(n + m - 1, n)
    assert perm.shape == (count,)
    cols = [j for j, c in enumerate(S) for _ in range(c)]
    rng = np.random.default_rng(n)
    if count <= 3000:
        outs = list(workloads.fock_outputs(m, n))
    picks = sorted({0, count - 1, *rng.integers(0, count, 25).tolist()})
    import paper_2403_04006_amd as pq
    for q in picks:
        T = outs[q] if count <= 3000 else pq.fock_unrank(m, n, q)
        if np.prod([int(t) + 1 for t in T]) > 20000:
            continue
        ref, size = permanent(U, cols, T), abs(permanent(np.abs(U), cols, T))
        assert abs(perm[q] - complex(ref)) <= 4 * n * EPS * float(size), (T, perm[q], ref)
        norm = math.exp(-0.5 * sum(math.lgamma(int(c) + 1.0) for c in [*S, *T]))
        assert abs(amp[q] - complex(ref) * norm) <= (4 * n + 200) * EPS * float(size) * norm
    if n <= 10:
        scale = np.abs(sweep).max()
        assert np.abs(perm - sweep).max() <= 1e-10 * scale
