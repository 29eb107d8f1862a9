"""Many EXTEND_ROW jobs on many modes: the plan's device memory follows the
columns that the jobs use, not the modes squared, and the outputs are those of
the same jobs in short lists."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MIB = 1 << 20


@pytest.mark.parametrize("m,pool", [
    (4096, 5),       # five columns: 320 KB of them, the whole matrix 256 MiB
    (4096, 512),     # 32 MiB of columns, the most that is transposed
    (4096, 513),     # one more: read from the matrix itself
])
def test_long_lists_on_many_modes(m, pool):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_04006_amd as pq
    rng = np.random.default_rng(pool)
    U = torch.from_numpy(rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m))).cuda() / np.sqrt(2 * m)
    cols = rng.permutation(m)[:pool]
    jobs = []
    for q in range(600):
        # every column of the pool in turn, three a job
        c = sorted(int(cols[(q + i) % pool]) for i in range(3))
        rows = sorted(rng.permutation(m)[:2].tolist())
        jobs.append({"op": pq.PQ_OP_EXTEND_ROW, "rows": [(i, 1) for i in rows], "cols": [(j, 1) for j in c], "out": q * m})
    eng = pq.Engine(0)
    out = torch.empty(600 * m, dtype=torch.complex128, device="cuda")
    eng.perm_many(U, jobs[:1], n_out=600 * m, with_amp=False, out=(out, None))
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    eng.perm_many(U, jobs, n_out=600 * m, with_amp=False, out=(out, None))
    torch.cuda.synchronize()
    used = free - torch.cuda.mem_get_info()[0]
    assert used <= 32 * MIB + 16 * MIB, used / MIB
    # the same bits as in lists of 300, which read U itself
    ref = torch.empty_like(out)
    for at in (0, 300):
        eng.perm_many(U, jobs[at:at + 300], n_out=600 * m, with_amp=False, out=(ref, None))
    torch.cuda.synchronize()
    assert torch.equal(out, ref)
    eng.close()
