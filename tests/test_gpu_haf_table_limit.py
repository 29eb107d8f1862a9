"""Tables of (loop) hafnians at the most photons that a pattern may have (64),
and one and two fewer, on few modes, in lists as long as the level-by-level form
needs to be the cheaper one, against the recursion over the last mode in 80-bit
arithmetic."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EPS = float(np.finfo(np.float64).eps)
LIST = 8000   # patterns that make a table of 64 photons the cheaper form


@pytest.fixture(scope="module")
def eng():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_04006_amd as pq
    return pq.Engine(0)


def recursion(A, gamma, caps):
    """h(r) for every r of at most `caps` photons: one photon of the last mode with itself, with another of its mode
    or with one of the modes before."""
    h = np.ones((1,), np.clongdouble)
    for k, cap in enumerate(caps):
        blocks = [h]
        for c in range(1, cap + 1):
            last = blocks[-1]
            v = gamma[k] * last
            if c >= 2:
                v = v + (c - 1) * A[k, k] * blocks[-2]
            base = 1
            for j in range(k):
                x, o = last.reshape(-1, caps[j] + 1, base), v.reshape(-1, caps[j] + 1, base)
                for e in range(1, caps[j] + 1):
                    o[:, e] += e * A[j, k] * x[:, e - 1]
                base *= caps[j] + 1
            blocks.append(v)
        h = np.concatenate(blocks)
    return h


def patterns(d, totals, caps, count):
    if d <= 3:
        return np.array([t for n in totals for t in workloads.fock_outputs(d, n)], np.int32)
    rng = np.random.default_rng(d)
    out = []
    while len(out) < count:
        r = rng.integers(0, np.array(caps) + 1)
        if int(r.sum()) in totals:
            out.append(r)
    return np.array(out, np.int32)


@pytest.mark.parametrize("loops", [False, True])
@pytest.mark.parametrize("totals", [(62,), (63,), (64,), (0, 2, 62, 63, 64)])
@pytest.mark.parametrize("d,cap", [(1, 64), (2, 64), (3, 64), (4, 20)])
def test_tables_up_to_64_photons(eng, d, cap, totals, loops):
    # the tolerance of the smaller tables: a level adds at most s + 3 roundings to a sum of products whose moduli add up
    # to the (loop) hafnian of the moduli
    rng = np.random.default_rng(100 * d + len(totals))
    A = 0.3 * (rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d)))
    A = np.triu(A) + np.triu(A, 1).T
    gamma = 0.5 * (rng.standard_normal(d) + 1j * rng.standard_normal(d)) if loops else None
    caps = [cap] * d
    reps = patterns(d, [n for n in totals if n <= d * cap], caps, 2500)
    reps = np.tile(reps, (-(-LIST // len(reps)), 1))
    got = eng.lhaf_many(torch.from_numpy(A).cuda(), None if gamma is None else torch.from_numpy(gamma).cuda(), reps)
    got = got.cpu().numpy()
    base = np.cumprod([1] + [cap + 1] * (d - 1))
    g = gamma if loops else np.zeros(d)
    ref = recursion(A, g, caps)[reps @ base]
    size = np.abs(recursion(np.abs(A), np.abs(g), caps)[reps @ base])
    N = reps.sum(1)
    bad = np.flatnonzero(np.abs(got - ref) > N * (N + 7) * EPS * size)
    assert bad.size == 0, (len(bad), reps[bad[0]], got[bad[0]], ref[bad[0]])


@pytest.mark.parametrize("loops", [False, True])
@pytest.mark.parametrize("reps", [[32, 32], [1, 63], [63, 1], [20, 44], [64, 0], [0, 64], [20, 0, 44], [1, 0, 63]])
def test_one_pattern_of_64_photons(eng, reps, loops):
    d = len(reps)
    rng = np.random.default_rng(sum(c * (i + 1) for i, c in enumerate(reps)))
    A = 0.3 * (rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d)))
    A = np.triu(A) + np.triu(A, 1).T
    gamma = 0.5 * (rng.standard_normal(d) + 1j * rng.standard_normal(d)) if loops else None
    out = eng.lhaf_many(torch.from_numpy(A).cuda(), None if gamma is None else torch.from_numpy(gamma).cuda(),
                        np.tile(np.array([reps], np.int32), (LIST, 1))).cpu().numpy()
    got = complex(out[0])
    assert np.array_equal(out, np.full_like(out, got))
    g = gamma if loops else np.zeros(d)
    ref = complex(recursion(A, g, reps)[-1])
    size = abs(complex(recursion(np.abs(A), np.abs(g), reps)[-1]))
    assert abs(got - ref) <= 64 * 71 * EPS * size, (reps, got, ref)
