"""EXTEND_ROW jobs on matrices whose columns differ in scale: every output is a
sum with one entry of every column, so the error follows the columns' scales as
the outputs do."""
import numpy as np
import pytest

import oracle
import workloads
from tests.tolerance import floor_of

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("powers", ["decades", "one large", "one small", "far apart", "zero column"])
@pytest.mark.parametrize("rows", [[1], [1] * 6, [2, 1, 3, 4], [1] * 12, [1] * 15, [1] * 17, [2] + [1] * 13])
def test_columns_of_different_scales(rows, powers):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_04006_amd as pq
    r, k = len(rows), sum(rows) + 1
    m = max(r, k) + 3
    rng = np.random.default_rng(k + 100 * r)
    cols = sorted(rng.permutation(m)[:k].tolist())
    scale = np.ones(m)
    if powers == "decades":
        scale = 10.0 ** rng.uniform(-3, 3, m)
    elif powers == "far apart":
        scale[cols[0]], scale[cols[-1]] = 1e100, 1e-100
    else:
        scale[cols[k // 2]] = {"one large": 10.0, "one small": 0.1, "zero column": 0.0}[powers]
    haar = workloads.haar(m, 70 + k)
    U = haar * scale
    modes = sorted(rng.permutation(m)[:r].tolist())
    job = {"op": pq.PQ_OP_EXTEND_ROW, "rows": list(zip(modes, rows)), "cols": [(c, 1) for c in cols]}
    eng = pq.Engine(0)
    out = eng.perm_many(torch.from_numpy(U).cuda(), [job], with_amp=False)[0].cpu().numpy()
    eng.close()
    drawn = [mo for mo, c in zip(modes, rows) for _ in range(c)]
    # (the oracle's own sums run over the columns' subsets: scaled after it)
    ref = oracle.extend_row(haar, drawn, cols) * np.prod(scale[cols])
    S = np.zeros(m, np.int32)
    S[cols] = 1
    for l in range(m):
        T = np.zeros(m, np.int32)
        np.add.at(T, drawn + [l], 1)
        assert abs(out[l] - ref[l]) <= max(1e-10 * abs(ref[l]), floor_of(U, S, T)), (l, out[l], ref[l])
