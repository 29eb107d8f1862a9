"""The calls that the engine's speed is judged by: what a photonic simulation has it do through its public entry points.

A case is a plain dict; `prepare` makes what a user's program holds before the call (matrices on the GPU, occupations
or job lists marshalled once), `run` makes one call, and `exact` gives the same outputs from the definitions in plain
torch and numpy, 64 bits throughout.

Kinds of call:
  perm       one amplitude <T|U|S>: unit occupations (boson sampling without collisions) or repeated ones
  batch      amplitudes of many repeated patterns of one interferometer
  replay     the marginals of a batch of chain-rule sampling runs (EXTEND_ROW jobs)
  mesh       one training step of a beamsplitter mesh: loss, interferometer and the angles' gradient
  grad       gradient of a few permanents with respect to U
  outputs    the amplitudes of every output of one input
  sample     boson samples drawn on the device, with or without loss
  lhaf       one (loop) hafnian with repeated modes
  table      the (loop) hafnians of every pattern of n photons in d modes
"""
import math

import numpy as np
import torch

import paper_2403_04006_amd as pq
from paper_2403_04006_amd import autograd

# ------------------------------------------------------------------- cases


def listed():
    return [
        # one amplitude of a small circuit, as called in a loop over outputs or circuits: latency
        {"name": "perm_small", "kind": "perm", "photons": 6, "modes": 12, "cap": 1},
        # one collision-free amplitude at the size where boson-sampling studies of a laptop end
        {"name": "perm_mid", "kind": "perm", "photons": 20, "modes": 40, "cap": 1},
        # the headline size of the benchmark: 30 photons, unit occupations
        {"name": "perm_large", "kind": "perm", "photons": 30, "modes": 120, "cap": 1},
        # the paper's permanent benchmark: every row and column repeated twice, odd number of modes
        {"name": "perm_repeated", "kind": "perm", "photons": 30, "modes": 15, "cap": 2},
        # a likelihood over measured patterns: 256 patterns of 40 photons in 20 modes, up to 4 in a mode
        {"name": "batch_repeated", "kind": "batch", "patterns": 256, "photons": 40, "modes": 20, "cap": 4},
        # marginals of 1000 sampling runs of 20 photons in 400 modes (19,000 jobs)
        {"name": "replay_20", "kind": "replay", "samples": 1000, "photons": 20, "modes": 400},
        # a training step: 12-mode rectangular mesh, 8 photons, 4096 measured outputs, forward and backward
        {"name": "mesh_step", "kind": "mesh", "modes": 12, "photons": 8, "patterns": 4096},
        # backward of one wide collision-free amplitude, an odd number of photons
        {"name": "grad_23", "kind": "grad", "photons": 23, "modes": 46, "cap": 1, "patterns": 1},
        # the full output state of 10 photons in 16 modes (3,268,760 amplitudes)
        {"name": "outputs_10_in_16", "kind": "outputs", "photons": 10, "modes": 16, "cap": 1},
        # 1000 boson samples of 20 photons in 400 modes, every draw on the device
        {"name": "sample_20", "kind": "sample", "samples": 1000, "photons": 20, "modes": 400, "lossy": False},
        # the loop hafnian of 18 displaced squeezed modes, two photons in each
        {"name": "lhaf_2x18", "kind": "lhaf", "modes": 18, "cap": 2, "loops": True},
        # a Gaussian boson sampling probability table: every pattern of 16 photons in 6 modes
        {"name": "table_16_in_6", "kind": "table", "photons": 16, "modes": 6, "loops": False},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """A case of the same kinds, its sizes over the whole range that the listed ones stand for."""
    kind = rng.choice(["perm", "perm", "batch", "replay", "mesh", "grad", "outputs", "sample", "lhaf", "table"])
    if kind == "perm":
        if rng.random() < 0.6:
            n = rng.randint(2, 31)
            return {"kind": kind, "photons": n, "modes": rng.randint(n, 4 * n), "cap": 1}
        m = rng.randint(3, 17)
        return {"kind": kind, "photons": rng.randint(m, 2 * m), "modes": m, "cap": rng.randint(2, 4)}
    if kind == "batch":
        m = rng.randint(4, 18)
        return {"kind": kind, "patterns": _log_int(rng, 4, 256), "photons": rng.randint(m, 2 * m), "modes": m,
                "cap": rng.randint(2, 4)}
    if kind == "replay":
        n = rng.randint(3, 20)
        return {"kind": kind, "samples": _log_int(rng, 10, 1000), "photons": n, "modes": _log_int(rng, max(n, 16), 400)}
    if kind == "mesh":
        m = rng.randint(4, 12)
        return {"kind": kind, "modes": m, "photons": rng.randint(2, min(8, m - 1)), "patterns": _log_int(rng, 16, 4096)}
    if kind == "grad":
        if rng.random() < 0.6:
            n = rng.randint(3, 25)
            return {"kind": kind, "photons": n, "modes": rng.randint(n, 3 * n), "cap": 1,
                    "patterns": _log_int(rng, 1, 64 if n <= 18 else 4)}
        m = rng.randint(3, 10)
        return {"kind": kind, "photons": rng.randint(m, 2 * m), "modes": m, "cap": rng.randint(2, 3),
                "patterns": _log_int(rng, 1, 64)}
    if kind == "outputs":
        while True:
            m, n = rng.randint(3, 20), rng.randint(2, 12)
            if math.comb(n + m - 1, n) <= 3_300_000:
                return {"kind": kind, "photons": n, "modes": m, "cap": 1 if n <= m and rng.random() < 0.6 else n}
    if kind == "sample":
        n = rng.randint(2, 20)
        return {"kind": kind, "samples": _log_int(rng, 1, 1000), "photons": n, "modes": _log_int(rng, max(n, 8), 400),
                "lossy": rng.random() < 0.4}
    if kind == "lhaf":
        return {"kind": kind, "modes": rng.randint(3, 18), "cap": 2 if rng.random() < 0.6 else 1,
                "loops": rng.random() < 0.5}
    while True:
        d, n = rng.randint(3, 9), 2 * rng.randint(1, 8)
        if math.comb(n + d - 1, n) <= 21_000:
            return {"kind": kind, "photons": n, "modes": d, "loops": rng.random() < 0.5}


# ------------------------------------------------------------------ inputs


def _haar(m, rng):
    z = rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m))
    q, r = np.linalg.qr(z)
    d = np.diagonal(r)
    return np.ascontiguousarray(q * (d / np.abs(d))[None, :])


def _occupations(rng, m, n, cap):
    """Uniform over the vectors of {0..cap}^m with sum n."""
    counts = [[1] + [0] * n]
    for _ in range(m):
        last = counts[-1]
        counts.append([sum(last[s - v] for v in range(min(cap, s) + 1)) for s in range(n + 1)])
    out, s = [0] * m, n
    for p in range(m, 0, -1):
        u = int(rng.random() * counts[p][s])
        for v in range(min(cap, s) + 1):
            if u < counts[p - 1][s - v] or v == min(cap, s):
                out[p - 1], s = v, s - v
                break
            u -= counts[p - 1][s - v]
    return out


def _cells(m):
    return tuple((k, k + 1) for col in range(m) for k in range(col % 2, m - 1, 2))


def _compositions(m, n):
    """Every vector of m counts with sum n, ascending lexicographically."""
    if m == 1:
        return np.full((1, 1), n, np.int32)
    blocks = []
    for v in range(n + 1):
        rest = _compositions(m - 1, n - v)
        blocks.append(np.concatenate([np.full((len(rest), 1), v, np.int32), rest], axis=1))
    return np.concatenate(blocks)


def _sparse(v):
    return [(i, int(c)) for i, c in enumerate(v) if c > 0]


def _inputs(case, seed):
    """The case's inputs as numpy arrays and lists, from the seed alone."""
    rng = np.random.default_rng([seed, 20240304])
    kind, m = case["kind"], case["modes"]
    x = {}
    if kind in ("perm", "batch", "grad"):
        count, n, cap = case.get("patterns", 1), case["photons"], case["cap"]
        x["U"] = _haar(m, rng)
        if kind == "perm" and cap == 2 and n == 2 * m:
            x["S"], x["T"] = [[2] * m], [[2] * m]
        else:
            x["S"] = [_occupations(rng, m, n, cap) for _ in range(count)]
            x["T"] = [_occupations(rng, m, n, cap) for _ in range(count)]
        if kind == "grad":
            x["g"] = rng.standard_normal(count) + 1j * rng.standard_normal(count)
    elif kind == "replay":
        x["U"] = _haar(m, rng)
        x["cols"] = [rng.permutation(case["photons"]).tolist() for _ in range(case["samples"])]
        x["rows"] = rng.integers(0, m, (case["samples"], case["photons"] - 1)).tolist()
    elif kind == "mesh":
        x["angles"] = rng.uniform(0.0, 2.0 * np.pi, (len(_cells(m)), 2))
        x["S"] = [1] * case["photons"] + [0] * (m - case["photons"])
        x["T"] = [_occupations(rng, m, case["photons"], 1) for _ in range(case["patterns"])]
    elif kind == "outputs":
        x["U"] = _haar(m, rng)
        x["S"] = _occupations(rng, m, case["photons"], case["cap"])
    elif kind == "sample":
        n = case["photons"]
        x["U"] = _haar(m, rng)
        x["order"] = np.stack([rng.permutation(n) for _ in range(case["samples"])]).astype(np.int32)
        x["uniforms"] = rng.random((case["samples"], n))
        x["eta"] = rng.uniform(0.8, 1.0, m).tolist() if case["lossy"] else None
    else:
        U = _haar(m, rng)
        x["A"] = np.ascontiguousarray((U * math.tanh(math.asinh(1.0))) @ U.T)
        x["gamma"] = 0.5 * (rng.standard_normal(m) + 1j * rng.standard_normal(m)) / math.sqrt(2.0)
        if kind == "lhaf":
            reps = [2] * m if case["cap"] == 2 else [1] * m
            if not case["loops"] and sum(reps) % 2:
                reps[0] += 1
            x["reps"] = reps
        else:
            x["reps"] = _compositions(m, case["photons"])
    return x


def _replay_jobs(x):
    jobs = []
    for cols, rows in zip(x["cols"], x["rows"]):
        counts = {}
        for k in range(2, len(cols) + 1):
            counts[rows[k - 2]] = counts.get(rows[k - 2], 0) + 1
            jobs.append({"op": pq.PQ_OP_EXTEND_ROW, "rows": sorted(counts.items()),
                         "cols": [(c, 1) for c in sorted(cols[:k])]})
    return jobs


def prepare(case, seed):
    x = _inputs(case, seed)
    dev = torch.device("cuda", torch.cuda.current_device())
    s = {"kind": case["kind"], "eng": pq.engine(dev.index), "m": case["modes"]}
    for k in ("U", "A", "gamma", "g", "order", "uniforms"):
        if k in x:
            s[k] = torch.from_numpy(x[k]).to(dev)
    kind = case["kind"]
    if kind == "perm":
        s["S"], s["T"] = x["S"][0], x["T"][0]
    elif kind == "batch":
        s["jobs"] = pq.JobSet([{"rows": _sparse(t), "cols": _sparse(c)} for c, t in zip(x["S"], x["T"])], s["m"])
    elif kind == "replay":
        s["jobs"] = pq.JobSet(_replay_jobs(x), s["m"])
    elif kind == "grad":
        s["pats"] = pq.PatternSet(x["S"], x["T"], s["m"])
    elif kind == "mesh":
        s["cells"] = _cells(s["m"])
        s["angles"] = torch.from_numpy(x["angles"]).to(dev).requires_grad_(True)
        s["pats"] = pq.PatternSet([x["S"]] * len(x["T"]), x["T"], s["m"])
    elif kind == "outputs":
        s["S"] = x["S"]
    elif kind == "sample":
        s["eta"] = x["eta"]
    else:
        s["gamma"] = s["gamma"] if case["loops"] else None
        s["reps"] = x["reps"]
    return s


# --------------------------------------------------------------------- run


def run(s):
    kind, eng = s["kind"], s["eng"]
    if kind == "perm":
        return eng.perm(s["U"], s["S"], s["T"])
    if kind == "batch":
        return eng.perm_batched(s["U"], s["jobs"])
    if kind == "replay":
        return eng.perm_many(s["U"], s["jobs"], with_amp=False)[0]
    if kind == "grad":
        return eng.grad_patterns(s["U"], s["pats"], s["g"], want_perm=True)
    if kind == "mesh":
        U = autograd.mesh_unitary(s["angles"], s["cells"], s["m"])
        loss = autograd.neg_log_prob(autograd.perm_amp(U, s["pats"]))
        (grad,) = torch.autograd.grad(loss, s["angles"])
        return {"U": U.detach(), "loss": loss.detach(), "grad": grad}
    if kind == "outputs":
        return eng.perm_all_outputs(s["U"], s["S"])
    if kind == "sample":
        if s["eta"] is not None:
            return eng.sample_chain_lossy(s["U"], s["eta"], s["order"], s["uniforms"])
        return eng.sample_chain(s["U"], s["order"], s["uniforms"])
    if kind == "lhaf":
        return eng.lhaf(s["A"], s["gamma"], s["reps"])
    return eng.lhaf_many(s["A"], s["gamma"], s["reps"])


# -------------------------------------------------------------------- work


def _terms(v):
    """Terms of the signed sum over the occupations v, one sign fixed."""
    v = [int(c) for c in v if c > 0]
    if not v:
        return 1
    lo = min(v)
    return math.prod(c + 1 for c in v) // (lo + 1) * lo


def _perm_flops(S, T):
    side, other = (S, T) if _terms(S) < _terms(T) else (T, S)
    c = sum(1 for v in other if v > 0)
    top = max(other, default=1)
    # per term: column sums moved by one row, the product of powers by grouped multiplies, the weighted sum
    return _terms(side) * (2.0 * c + 6.0 * (c + top - 2) + 4.0)


def work(case):
    """Bytes: inputs once, outputs once.  Flops: the sums over sign vectors that the definitions reduce to, or the
    recursion photon by photon where that is cheaper."""
    kind, m = case["kind"], case["modes"]
    n = case.get("photons", 0)
    if kind in ("perm", "batch", "grad"):
        x = _inputs({**case, "patterns": min(case.get("patterns", 1), 8)}, 0)
        count = case.get("patterns", 1)
        flops = sum(_perm_flops(a, b) for a, b in zip(x["S"], x["T"])) / len(x["S"]) * count
        # a gradient takes every leave-one-out product: about three times the multiplies
        return {"bytes": 16.0 * m * m * (2 if kind == "grad" else 1) + 32.0 * count, "flops": flops * (3 if kind == "grad" else 1)}
    if kind in ("replay", "sample"):
        per = sum(2.0 ** max(0, k - 2) * (18.0 * k) + 8.0 * k * m for k in range(2, n + 1))
        out = 16.0 * m * (n - 1) if kind == "replay" else 4.0 * n
        return {"bytes": case["samples"] * (out + 12.0 * n) + 16.0 * m * m, "flops": case["samples"] * per}
    if kind == "mesh":
        distinct = min(case["patterns"], math.comb(m, n))
        return {"bytes": 16.0 * len(_cells(m)) * 2 + 32.0 * m * m + 16.0 * case["patterns"],
                "flops": 4.0 * distinct * 2.0 ** (n - 1) * (8.0 * n - 4.0)}
    if kind == "outputs":
        # photon by photon: every amplitude is a sum over its occupied modes of the one-photon-less amplitudes
        flops = sum(8.0 * math.comb(k + m - 1, k) * min(k, m) for k in range(1, n + 1))
        return {"bytes": 16.0 * m * m + 32.0 * math.comb(n + m - 1, n), "flops": flops}
    if kind == "lhaf":
        t = _terms([case["cap"]] * m)
        return {"bytes": 16.0 * m * m + 16.0, "flops": t * (200.0 if case["loops"] else 65.0)}
    # table: the recursion over all patterns of fewer photons
    count = math.comb(n + m - 1, n)
    return {"bytes": 16.0 * m * m + 16.0 * count + 4.0 * m * count,
            "flops": 8.0 * m * sum(math.comb(k + m - 1, k) for k in range(0, n + 1, 1 if case["loops"] else 2))}


# ------------------------------------------------------------------- exact

_CHUNK = 1 << 21


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _most_terms():
    return 2_000_000_000 if torch.cuda.is_available() else 2_000_000


def _sign_sums(B, mu, dev):
    """Chunks (w, delta, c) of the signed sum over rows with multiplicities mu (one copy of the rarest row fixed):
    weights, the rows' delta values and the column sums."""
    f = int(np.argmin(mu))
    radix = [int(c) if i == f else int(c) + 1 for i, c in enumerate(mu)]
    total = math.prod(radix)
    Bt = torch.from_numpy(np.ascontiguousarray(B)).to(dev)
    for a in range(0, total, _CHUNK):
        rank = torch.arange(a, min(total, a + _CHUNK), device=dev)
        w = torch.ones(len(rank), dtype=torch.float64, device=dev)
        delta = torch.empty((len(mu), len(rank)), dtype=torch.float64, device=dev)
        for i, rho in enumerate(radix):
            d = rank % rho
            rank = rank // rho
            binom = torch.tensor([(-1.0) ** k * math.comb(rho - 1, k) for k in range(rho)], dtype=torch.float64, device=dev)
            w = w * binom[d]
            delta[i] = float(mu[i]) - 2.0 * d.to(torch.float64)
        c = torch.complex(Bt.real.T.contiguous() @ delta, Bt.imag.T.contiguous() @ delta)
        yield w, delta, c


def _perm(U, S, T, grad=False):
    """perm(U_{T,S}), and with grad its derivative with respect to U."""
    rows, cols = _sparse(T), _sparse(S)
    flip = _terms(S) < _terms(T)
    if flip:
        rows, cols = cols, rows
    M = U.T if flip else U
    dev = _device()
    n = sum(c for _, c in rows)
    B = M[np.ix_([i for i, _ in rows], [j for j, _ in cols])]
    mu, kap = [c for _, c in rows], [c for _, c in cols]
    value = torch.zeros((), dtype=torch.complex128, device=dev)
    D = torch.zeros((len(mu), len(kap)), dtype=torch.complex128, device=dev)
    for w, delta, c in _sign_sums(B, mu, dev):
        if not grad:
            p = w.to(torch.complex128)
            for j, k in enumerate(kap):
                for _ in range(k):
                    p = p * c[j]
            value += p.sum()
            continue
        pre = [w.to(torch.complex128)]
        for j, k in enumerate(kap):
            y = pre[-1]
            for _ in range(k):
                y = y * c[j]
            pre.append(y)
        value += pre[-1].sum()
        suf = torch.ones_like(pre[0])
        for j in reversed(range(len(kap))):
            g = pre[j] * suf * kap[j]
            for _ in range(kap[j] - 1):
                g = g * c[j]
                suf = suf * c[j]
            suf = suf * c[j]
            D[:, j] += torch.complex(delta @ g.real, delta @ g.imag)
    scale = 2.0 ** -(n - 1)
    out = complex(value) * scale
    if not grad:
        return out
    full = np.zeros(M.shape, complex)
    full[np.ix_([i for i, _ in rows], [j for j, _ in cols])] = D.cpu().numpy() * scale
    return out, (full.T if flip else full)


def _norm(S, T):
    return math.exp(-0.5 * sum(math.lgamma(int(c) + 1.0) for c in list(S) + list(T)))


def _exact_replay(x, m):
    dev = _device()
    U = torch.from_numpy(x["U"]).to(dev)
    outs = []
    for cols, rows in zip(x["cols"], x["rows"]):
        for k in range(2, len(cols) + 1):
            drawn, c = rows[: k - 1], sorted(cols[:k])
            L = torch.zeros(k, dtype=torch.complex128, device=dev)
            for w, _, s in _sign_sums(x["U"][np.ix_(drawn, c)], [1] * (k - 1), dev):
                pre, suf = [w.to(torch.complex128)], torch.ones_like(s[0])
                for j in range(k - 1):
                    pre.append(pre[-1] * s[j])
                for j in reversed(range(k)):
                    L[j] += (pre[j] * suf).sum()
                    suf = suf * s[j]
            outs.append((U[:, c] * (L * 2.0 ** -(k - 2))[None, :]).sum(1))
    return torch.cat(outs)


def _exact_mesh(x, case):
    m, n = case["modes"], case["photons"]
    a = torch.from_numpy(x["angles"]).requires_grad_(True)
    U = torch.eye(m, dtype=torch.complex128)
    for k, (i, j) in enumerate(_cells(m)):
        t = torch.cos(a[k, 0]).to(torch.complex128)
        r = torch.polar(torch.sin(a[k, 0]), a[k, 1]) if torch.sin(a[k, 0]) >= 0 else -torch.polar(-torch.sin(a[k, 0]), a[k, 1])
        rows = list(U.unbind(0))
        rows[i], rows[j] = t * U[i] - r.conj() * U[j], r * U[i] + t * U[j]
        U = torch.stack(rows)
    pats, back = np.unique(np.array(x["T"]), axis=0, return_inverse=True)
    back = torch.from_numpy(back.reshape(-1))
    idx = torch.from_numpy(np.stack([np.flatnonzero(p) for p in pats]))
    sub = U[idx][:, :, :n]                                            # pattern, row, column
    perm = torch.zeros(len(pats), dtype=torch.complex128)
    for d in range(2 ** (n - 1)):
        delta = torch.tensor([1.0] + [-1.0 if d >> i & 1 else 1.0 for i in range(n - 1)], dtype=torch.float64)
        perm = perm + delta.prod() * (delta[None, :, None] * sub).sum(1).prod(1)
    perm = perm * 2.0 ** -(n - 1)
    loss = -(torch.log(perm.real.square() + perm.imag.square())[back]).mean()
    (grad,) = torch.autograd.grad(loss, a)
    return {"U": U.detach(), "loss": loss.detach(), "grad": grad}


def _exact_outputs(U, S, m):
    """Photon by photon: amplitudes of k photons from those of k - 1."""
    dev = _device()
    n = int(sum(S))
    modes = [j for j, c in enumerate(S) for _ in range(c)]
    Ut = torch.from_numpy(U).to(dev)

    def step(q, rem, v):   # vectors that start with a smaller count than v in the first of q + 1 places
        return sum(math.comb(rem - u + q - 1, q - 1) for u in range(v)) if q else 0

    value = torch.ones(1, dtype=torch.complex128, device=dev)
    T = None
    for k in range(1, n + 1):
        T = torch.from_numpy(_compositions(m, k)).to(dev).to(torch.int64)
        tabs = [torch.tensor([[step(m - 1 - i, r, min(v, r)) for v in range(k + 1)] for r in range(k + 1)], device=dev)
                for i in range(m)]
        out = torch.zeros(len(T), dtype=torch.complex128, device=dev)
        for i in range(m):
            has = torch.nonzero(T[:, i] > 0).reshape(-1)
            X = T[has].clone()
            X[:, i] -= 1
            rem = torch.full((len(has),), k - 1, dtype=torch.int64, device=dev)
            rank = torch.zeros_like(rem)
            for p in range(m - 1):
                rank += tabs[p][rem, X[:, p]]
                rem -= X[:, p]
            out[has] += T[has, i].to(torch.float64) * Ut[i, modes[k - 1]] * value[rank]
        value = out
    norm = torch.exp(-0.5 * (torch.lgamma(T.to(torch.float64) + 1.0).sum(1) + sum(math.lgamma(c + 1.0) for c in S)))
    return [value, value * norm]


def _exact_hafnians(A, gamma, reps):
    """Loop hafnians by the recursion over the first occupied mode, over all smaller patterns."""
    reps = np.asarray(reps, np.int64).reshape(-1, A.shape[0])
    d = A.shape[0]
    top = reps.max(0)
    base = np.concatenate([[1], np.cumprod(top + 1)[:-1]]).astype(np.int64)
    size = int(np.prod(top + 1))
    grid = np.stack([(np.arange(size) // base[i]) % (top[i] + 1) for i in range(d)], 1)
    total = grid.sum(1)
    A = np.triu(A) + np.triu(A, 1).T
    h = np.zeros(size, complex)
    h[0] = 1.0
    for s in range(1, int(reps.sum(1).max()) + 1):
        at = np.flatnonzero(total == s)
        first = (grid[at] > 0).argmax(1)
        less = at - base[first]
        v = gamma[first] * h[less] if gamma is not None else np.zeros(len(at), complex)
        rest = grid[less]
        for k in range(d):
            ok = rest[:, k] > 0
            v[ok] += rest[ok, k] * A[first[ok], k] * h[less[ok] - base[k]]
        h[at] = v
    return h[reps @ base]


def _exact_lhaf(A, gamma, reps, loops):
    if np.prod([c + 1.0 for c in reps]) <= 3e6:
        return _exact_hafnians(A, gamma if loops else None, [reps])
    if _terms(reps) > _most_terms() / 4:
        return None
    # too many smaller patterns: the signed sum over vertices
    dev = _device()
    A = np.triu(A) + np.triu(A, 1).T
    N = int(sum(reps))
    g = torch.from_numpy(gamma).to(dev)
    total = torch.zeros((), dtype=torch.complex128, device=dev)
    for w, X, AX in _sign_sums(A, list(reps), dev):
        x = 0.5 * (AX * X).sum(0)
        if not loops:
            p = x ** (N // 2) / math.factorial(N // 2)
        else:
            l = torch.complex(g.real @ X, g.imag @ X)
            odd, y = N % 2, l * l
            # sum_j x^j l^(N - 2j) / (j! (N - 2j)!), Horner-like over j from the smallest power of l
            p, powers = torch.zeros_like(x), [torch.ones_like(x)]
            for _ in range(N // 2):
                powers.append(powers[-1] * x)
            ly = torch.ones_like(x)
            for j in range(N // 2, -1, -1):
                p = p + powers[j] * ly / float(math.factorial(j) * math.factorial(N - 2 * j))
                ly = ly * y
            p = p * l if odd else p
        total += (w * p).sum()
    return np.array([complex(total) * 2.0 ** -(N - 1)])


def exact(case, seed):
    kind, m = case["kind"], case["modes"]
    if kind == "sample":
        return None
    x = _inputs(case, seed)
    if kind in ("perm", "batch", "grad"):
        total = sum(min(_terms(a), _terms(b)) for a, b in zip(x["S"], x["T"]))
        if total > _most_terms() // (8 if kind == "grad" else 1) or len(x["S"]) > 64:
            return None
        if kind == "grad":
            dU, perms = np.zeros((m, m), complex), []
            for a, b, g in zip(x["S"], x["T"], x["g"]):
                p, D = _perm(x["U"], a, b, grad=True)
                perms.append(p)
                dU += g * D.conj()
            return [dU, np.array(perms)]
        perms = np.array([_perm(x["U"], a, b) for a, b in zip(x["S"], x["T"])])
        amps = perms * np.array([_norm(a, b) for a, b in zip(x["S"], x["T"])])
        return [perms[0], amps[0]] if kind == "perm" else [perms, amps]
    if kind == "replay":
        return _exact_replay(x, m) if case["samples"] * case["photons"] <= 1000 else None
    if kind == "mesh":
        return _exact_mesh(x, case)
    if kind == "outputs":
        return _exact_outputs(x["U"], x["S"], m)
    if kind == "lhaf":
        return _exact_lhaf(x["A"], x["gamma"], x["reps"], case["loops"])
    return _exact_hafnians(x["A"], x["gamma"] if case["loops"] else None, x["reps"])
