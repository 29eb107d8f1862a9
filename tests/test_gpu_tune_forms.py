"""Recorded autotuning decisions on the forms of the later kernels: a recorded
policy sets the chunks of EXTEND_ROW jobs swept over column signs."""
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
