"""EXTEND_ROW jobs over the signs of their columns in perm_batched: the bits of
the static schedule at the edges of their classes in every queue mode, and the
host's request to stop."""
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


def extend_jobs(pq, m, count, rows, cols, seed):
    """`count` jobs of that many drawn rows (all different) and columns."""
    rng = np.random.default_rng(seed)
    return [{"op": pq.PQ_OP_EXTEND_ROW, "rows": [(i, 1) for i in sorted(rng.permutation(m)[:rows].tolist())],
             "cols": [(c, 1) for c in sorted(rng.permutation(m)[:cols].tolist())]} for _ in range(count)]


@pytest.mark.parametrize("k", [4, 9, 12, 13, 14, 17, 19, 22, 24])
def test_every_queue_mode_gives_the_static_bits(pq, k):
    # every column class, from single-chunk jobs to 2^9 chunks a job, beside short jobs of one other class and a
    # permanent
    m = 26
    eng = pq.Engine(0)
    U = torch.from_numpy(workloads.haar(m, k)).cuda()
    jobs = extend_jobs(pq, m, 6 if k > 20 else 40, k - 1, k, k) + extend_jobs(pq, m, 5, 15, 16, 1)
    jobs.append({"op": pq.PQ_OP_PERM, "rows": [(i, 1) for i in range(18)], "cols": [(i, 1) for i in range(18)]})
    ref = eng.perm_many(U, jobs, with_amp=False)[0].cpu().numpy()
    for mode in ("always", "auto", "never"):
        eng.queue_mode(mode)
        for _ in range(3):   # the captured graph's replays, with eager work between
            got = eng.perm_batched(U, jobs, with_amp=False)[0].cpu().numpy()
            assert np.array_equal(got, ref), mode
    eng.close()


@pytest.mark.parametrize("mode", ["auto", "always"])
def test_cancel_stops_long_extend_row_jobs(pq, mode):
    m = 30
    eng = pq.Engine(0)
    eng.queue_mode(mode)
    U = torch.from_numpy(workloads.haar(m, 3)).cuda()
    jobs = pq.JobSet(extend_jobs(pq, m, 400, 23, 24, 5), m)
    n = 400 * m
    full = eng.perm_many(U, jobs, with_amp=False)[0]
    out = torch.zeros(n, dtype=torch.complex128, device="cuda")
    eng.perm_batched(U, jobs, with_amp=False, out=(out, None))
    torch.cuda.synchronize()
    assert torch.equal(out, full)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    eng.perm_batched(U, jobs, with_amp=False, out=(out, None))
    e1.record()
    torch.cuda.synchronize()
    t_full = e0.elapsed_time(e1)
    e0.record()
    eng.perm_batched(U, jobs, with_amp=False, out=(out, None))
    eng.cancel(True)
    e1.record()
    torch.cuda.synchronize()
    t_cut = e0.elapsed_time(e1)
    print(f"queue: {t_full:.2f} ms, cancelled: {t_cut:.2f} ms", flush=True)
    assert t_cut < 0.8 * t_full
    eng.cancel(False)
    eng.perm_batched(U, jobs, with_amp=False, out=(out, None))
    torch.cuda.synchronize()
    assert torch.equal(out, full)
    eng.close()
