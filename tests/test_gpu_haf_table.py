"""Tables of (loop) hafnians built level by level (pq_lhaf_many on many
patterns of few modes) against the oracle, at the edges of the level sizes,
photon groups and pattern lists."""
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


def table(d, totals):
    return np.array([t for n in totals for t in workloads.fock_outputs(d, n)], np.int32)


@pytest.mark.parametrize("loops", [False, True])
@pytest.mark.parametrize("d,totals,unused", [
    (1, range(0, 9), 0),            # one mode: one vector a level
    (2, (1, 2), 1),                 # an unoccupied mode; without loops a single level
    (4, (5, 6), 0),                 # odd patterns are zero without loops
    (5, (0, 3, 8), 2),              # trivial patterns beside others; two unoccupied modes
    (5, (10,), 0),                  # groups of four photons and a rest
    (6, (8, 10), 0),                # level 9 (2002 vectors) in the small kernel, 10 (3003) not
])
def test_table_matches_oracle(eng, d, totals, unused, loops):
    # a level adds at most s + 3 roundings to a sum of products whose moduli
    # add up to the (loop) hafnian of the moduli: N (N + 7) eps of it in all
    m = d + unused
    rng = np.random.default_rng(7 * d + unused)
    A = rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m))   # not symmetric: the upper triangle counts
    gamma = workloads.loop_vector(m, d) if loops else None
    reps = np.zeros((0, m), np.int32)
    occupied = sorted(rng.permutation(m)[:d])
    reps = np.zeros((len(table(d, totals)), m), np.int32)
    reps[:, occupied] = table(d, totals)
    reps = reps[rng.permutation(len(reps))]
    got = eng.lhaf_many(torch.from_numpy(A).cuda(), None if gamma is None else torch.from_numpy(gamma).cuda(), reps)
    got = got.cpu().numpy()
    Au = np.triu(A) + np.triu(A, 1).T
    for q in rng.permutation(len(reps))[:60]:
        r, N = reps[q], int(reps[q].sum())
        ref = oracle.lhaf_rep(Au, gamma, r)
        size = abs(oracle.lhaf_rep(np.abs(Au).astype(complex), None if gamma is None else np.abs(gamma).astype(complex), r))
        assert abs(got[q] - ref) <= N * (N + 7) * EPS * size, (r, got[q], ref)


def test_table_of_many_modes(eng):
    # 32 modes, the most of this form: four photons against single hafnians
    A = torch.from_numpy(workloads.gbs_matrix(32, 3)).cuda()
    rng = np.random.default_rng(9)
    reps = np.stack([np.bincount(rng.integers(0, 32, 4), minlength=32) for _ in range(3000)]).astype(np.int32)
    reps[:32, :] = 2 * np.eye(32, dtype=np.int32)                        # every mode occupied
    got = eng.lhaf_many(A, None, reps).cpu().numpy()
    for q in [0, 31, *rng.integers(32, 3000, 30).tolist()]:
        one = complex(eng.lhaf(A, None, reps[q]).item())
        assert abs(got[q] - one) <= 1e-13, (reps[q], got[q], one)


def test_table_refuses_what_the_sweeps_refuse(eng):
    import paper_2403_04006_amd as pq
    A = torch.from_numpy(workloads.gbs_matrix(4, 0)).cuda()
    good = np.tile(np.array([[1, 1, 0, 0]], np.int32), (300, 1))
    for bad in ([1, -1, 0, 0], [65, 1, 0, 0], [33, 32, 0, 0], [2**31 - 1, 1, 0, 0], [128, 128, 0, 0]):
        reps = np.concatenate([good, np.array([bad], np.int32)])
        with pytest.raises(pq.PqError):
            eng.lhaf_many(A, None, reps)
