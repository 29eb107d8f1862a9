"""Recorded autotuning decisions on the forms of the later kernels: a recorded
policy sets the chunks of EXTEND_ROW jobs swept over column signs, and short
permanents have the one-launch form among their candidates."""
import json

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_04006_amd as pq
    return pq


def rewrite(path, policy):
    """The one recorded decision with another policy."""
    (line,) = path.read_text().strip().splitlines()
    rec = json.loads(line)
    rec["policy"] = list(policy)
    path.write_text(json.dumps(rec) + "\n")


def test_a_recorded_policy_sets_the_chunks_of_column_signs(pq, tmp_path, monkeypatch):
    # 40 jobs of 22 columns: 2^21 terms each, 2^15 time states; chunks of 256, 64 and 32 states give the same sums in
    # another order of rounding
    m = 24
    rng = np.random.default_rng(2)
    jobs = [{"op": pq.PQ_OP_EXTEND_ROW, "rows": [(i, 1) for i in sorted(rng.permutation(m)[:21].tolist())],
             "cols": [(c, 1) for c in sorted(rng.permutation(m)[:22].tolist())]} for _ in range(40)]
    U = torch.from_numpy(workloads.haar(m, 5)).cuda()
    plain = pq.Engine(0)
    want = plain.perm_many(U, jobs, with_amp=False)[0].cpu().numpy()
    plain.close()
    path = tmp_path / "tune.jsonl"
    monkeypatch.setenv("PQ_AUTOTUNE_CACHE", str(path))
    monkeypatch.setenv("PQ_AUTOTUNE", "1")
    first = pq.Engine(0)
    first.perm_many(U, jobs, with_amp=False)
    assert first.autotune_last()["candidates"] == 14
    first.close()
    got = {}
    for policy in ((64, 8, 256), (64, 64, 64), (64, 64, 32)):
        rewrite(path, policy)
        eng = pq.Engine(0)
        got[policy] = eng.perm_many(U, jobs, with_amp=False)[0].cpu().numpy()
        info = eng.autotune_last()
        assert info["candidates"] == 0 and (info["waves_per_cu"], info["chunks_per_wave"], info["min_chunk"]) == policy
        eng.close()
    a, b, c = got.values()
    assert np.array_equal(a, want)                                  # the default policy, recorded or not
    assert not np.array_equal(a, b) and not np.array_equal(b, c)
    scale = np.abs(a).max()
    assert np.abs(a - b).max() <= 1e-12 * scale and np.abs(a - c).max() <= 1e-12 * scale


@pytest.mark.parametrize("S,T", [
    ([1] * 20, [1] * 20),                              # binary digits
    ([2] * 9, [2] * 9),                                # mixed radices
])
def test_short_permanents_tune_the_one_launch_form(pq, tmp_path, monkeypatch, S, T):
    # a record of 0 wavefronts is the default's one launch, bit for bit; another one the longer sequence
    m = len(S)
    U = torch.from_numpy(workloads.haar(m, 4)).cuda()
    plain = pq.Engine(0)
    want = complex(plain.perm(U, S, T)[0].item())
    plain.close()
    path = tmp_path / "tune.jsonl"
    monkeypatch.setenv("PQ_AUTOTUNE_CACHE", str(path))
    monkeypatch.setenv("PQ_AUTOTUNE", "1")
    first = pq.Engine(0)
    tuned = complex(first.perm(U, S, T)[0].item())
    info = first.autotune_last()
    first.close()
    assert info["candidates"] == 3 and info["best_ms"] <= info["default_ms"]
    assert abs(tuned - want) <= 1e-12 * abs(want)
    if info["waves_per_cu"] == 0:
        assert tuned == want
    got = {}
    for waves in (0, 4):
        rewrite(path, (waves, 1, 32))
        eng = pq.Engine(0)
        got[waves] = complex(eng.perm(U, S, T)[0].item())
        assert eng.autotune_last()["candidates"] == 0 and eng.autotune_last()["waves_per_cu"] == waves
        # the allocation-free call follows the record
        out = torch.empty(1, dtype=torch.complex128, device="cuda")
        occ = [(pq._lib.ctypes.c_int32 * m)(*v) for v in (S, T)]
        torch.cuda.synchronize()
        assert eng._lib.pq_perm_noalloc(eng._ctx, U.data_ptr(), U.stride(0), m, occ[0], occ[1], out.data_ptr(), None,
                                        torch.cuda.current_stream().cuda_stream) == 0
        assert complex(out.item()) == got[waves]
        eng.close()
    assert got[0] == want
    assert got[4] != want and abs(got[4] - want) <= 1e-12 * abs(want)
