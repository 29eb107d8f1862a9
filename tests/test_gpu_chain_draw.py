"""The device sampler's draw at targets that rounding puts between the prefix
sums of its 64 lanes: the mode drawn always has a weight, also where a lane of
zero weights is the first whose sum exceeds the target."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MODES = 64   # one mode a lane


@pytest.fixture(scope="module")
def eng():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_04006_amd as pq
    return pq.Engine(0)


def scan(w):
    """Inclusive prefix sums over 64 lanes, by doubling distances."""
    upto = w.copy()
    for h in (1, 2, 4, 8, 16, 32):
        o = np.concatenate([np.zeros(h), upto[:-h]])
        upto = np.where(np.arange(MODES) >= h, upto + o, upto)
    return upto


def uniform_for(lo, hi, total):
    """A uniform u with lo <= fl(u * total) < hi, or None."""
    u = lo / total
    for _ in range(4):
        if lo <= u * total < hi and u < 1.0:
            return u
        u = np.nextafter(u, 2.0 if u * total < lo else 0.0)
    return None


def cases(seed):
    """One column of real amplitudes, and uniforms whose target lies where the first lane beyond it has no weight, or
    where none beyond it has."""
    rng = np.random.default_rng(seed)
    x = rng.random(MODES) * (rng.random(MODES) < 0.5)
    x[-rng.integers(1, 4):] = 0.0
    w = x * x
    upto = scan(w)
    total, last = upto[-1], int(np.flatnonzero(w).max())
    us, want = [], []
    for z in range(1, MODES):
        before = upto[:z].max()
        if w[z] == 0.0 and upto[z] > before:
            u = uniform_for(before, upto[z], total)
            if u is not None:
                us.append(u)
                # the neighbours of positive weight
                want.append({int(l) for l in np.flatnonzero(w[:z])[-1:]} | {int(l) + z for l in np.flatnonzero(w[z:])[:1]})
    assert last < MODES - 1
    return x, us, want


def test_draws_have_a_weight(eng):
    found = 0
    for seed in range(400):
        x, us, want = cases(seed)
        if not us:
            continue
        U = torch.zeros((MODES, MODES), dtype=torch.complex128)
        U[:, 0] = torch.from_numpy(x)
        out = eng.sample_chain(U.cuda(), torch.zeros((len(us), 1), dtype=torch.int32).cuda(),
                               torch.tensor(us, dtype=torch.float64).reshape(-1, 1).cuda()).cpu().numpy().reshape(-1)
        for pick, ok, u in zip(out.tolist(), want, us):
            assert x[pick] > 0.0 and pick in ok, (seed, pick, ok, u)
        found += len(us)
    assert found >= 50


def test_draws_without_a_weight_keep_the_last_mode(eng):
    # nothing to draw from, and a uniform of one: the last mode, as before
    U = torch.zeros((MODES, MODES), dtype=torch.complex128)
    order = torch.zeros((1, 1), dtype=torch.int32).cuda()
    assert int(eng.sample_chain(U.cuda(), order, torch.tensor([[0.5]], dtype=torch.float64).cuda())) == MODES - 1
    U[3, 0] = 1.0
    assert int(eng.sample_chain(U.cuda(), order, torch.tensor([[1.0]], dtype=torch.float64).cuda())) == MODES - 1
    assert int(eng.sample_chain(U.cuda(), order, torch.tensor([[0.0]], dtype=torch.float64).cuda())) == 3
    U[9, 0] = complex(np.nan, 0.0)
    assert int(eng.sample_chain(U.cuda(), order, torch.tensor([[0.5]], dtype=torch.float64).cuda())) == MODES - 1
