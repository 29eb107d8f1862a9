"""The device sampler at the edges of its row counts and wavefront splits:
draws against the oracle's, and both splits against each other."""
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


@pytest.mark.parametrize("n,m", [
    (1, 1), (2, 2), (3, 70),     # no, one, two signs; more modes than lanes
    (7, 7), (8, 65),             # all signs on lanes; the first wavefront column
    (9, 12), (10, 13),           # the last size of the 8-row kernel, the first of the 12-row one
    (11, 11), (12, 130),         # one and two time columns
    (13, 20), (14, 20),          # three and four; 12 rows and 16
])
@pytest.mark.parametrize("samples", [256, 257])   # eight and four wavefronts a sample
def test_draws_match_oracle(eng, n, m, samples):
    U = workloads.haar(m, 300 + n)
    rng = np.random.default_rng(n)
    # the input modes, one of them repeated where there are two
    inputs = rng.permutation(m)[:n]
    if n > 1:
        inputs[1] = inputs[0]
    order = np.stack([rng.permutation(inputs) for _ in range(samples)]).astype(np.int32)
    u = rng.random((samples, n))
    u[0] = 0.0
    u[1] = np.nextafter(1.0, 0.0)
    out = eng.sample_chain(torch.from_numpy(U).cuda(), torch.from_numpy(order), torch.from_numpy(u)).cpu().numpy()
    assert out.min() >= 0 and out.max() < m
    for s in [2, 3, samples // 2, samples - 1]:
        rows, margins = oracle.chain_rule_sample(U, list(order[s]), u[s])
        for k in range(n):
            if out[s, k] != rows[k]:
                assert margins[k] < 1e-9, (s, k, margins[k])
                break


@pytest.mark.parametrize("n", [17, 18, 21, 22, 24])
def test_both_splits_draw_the_same(eng, n):
    m = 60
    U = torch.from_numpy(workloads.haar(m, n)).cuda()
    rng = np.random.default_rng(n)
    order = torch.from_numpy(np.stack([rng.permutation(n) for _ in range(260)]).astype(np.int32))
    u = torch.from_numpy(rng.random((260, n)))
    wide = eng.sample_chain(U, order[:8], u[:8])
    both = eng.sample_chain(U, order, u) if n < 24 else eng.sample_chain(U, order[:8].repeat(33, 1), u[:8].repeat(33, 1))
    assert torch.equal(both[:8], wide)
