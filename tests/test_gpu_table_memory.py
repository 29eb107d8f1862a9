"""The forms that build tables in workspace, where there is no memory for the
table: the call goes on in the form that needs none."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture()
def eng():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_04006_amd as pq
    eng = pq.Engine(0)
    yield eng
    eng.close()


def test_all_outputs_without_memory_for_the_levels(eng):
    import paper_2403_04006_amd as pq
    m, n = 16, 8                                   # 3.4 MB of lower levels; the sweep's workspace is within 1 MB
    U = torch.from_numpy(workloads.haar(m, 1)).cuda()
    S = [1] * n + [0] * (m - n)
    eng.all_outputs_gemm("never")
    sweep = eng.perm_all_outputs(U, S)
    eng.all_outputs_gemm("auto")
    eng.fault_inject(pq._lib.PQ_FAULT_ALLOC)
    got = eng.perm_all_outputs(U, S)
    eng.fault_inject(pq._lib.PQ_FAULT_NONE)
    assert all(torch.equal(a, b) for a, b in zip(got, sweep))
    levels = eng.perm_all_outputs(U, S)            # with memory again
    assert float((levels[0] - sweep[0]).abs().max()) <= 1e-13 and not torch.equal(levels[0], sweep[0])


def test_hafnian_table_without_memory_for_it(eng):
    import paper_2403_04006_amd as pq
    m, d, n = 40, 12, 14                           # 4.5 million vectors of 14 photons in 12 modes, 100 MB of even levels
    A = torch.from_numpy(workloads.gbs_matrix(m, 2)).cuda()
    rng = np.random.default_rng(3)

    def patterns(modes, count):
        return np.stack([np.bincount(rng.integers(0, modes, n), minlength=m) for _ in range(count)]).astype(np.int32)

    few = patterns(d, 3000)
    other = pq.Engine(0)
    table = other.lhaf_many(A, None, few)
    torch.cuda.synchronize()
    other.close()
    wide = patterns(m, 6000)                       # too many modes for a table: workspace of the sweeps
    eng.lhaf_many(A, None, wide)
    eng.fault_inject(pq._lib.PQ_FAULT_ALLOC)
    got = eng.lhaf_many(A, None, few)
    eng.fault_inject(pq._lib.PQ_FAULT_NONE)
    torch.cuda.synchronize()
    assert float((got - table).abs().max()) <= 1e-12
    assert not torch.equal(got, table)
    assert torch.equal(eng.lhaf_many(A, None, few), table)   # with memory again
