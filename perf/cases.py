"""Performance cases of the local-energy path: what a VMC program, a batch of
small molecules, a service and a non-molecular Hamiltonian ask of the library,
through its public entry points.

A case names a Hamiltonian, a batch of samples and the entry point.  The
Hamiltonians are this repository's synthetic molecules (workloads: integrals
decaying with the orbital distance, Jordan-Wigner strings) and one table
outside the molecular form.  A Hamiltonian and its resident handle are built
once per process and shared by every state, as in a program that optimises
one molecule: each step brings new samples in new buffers to the same handle.

Samples: occupied orbitals are the n largest of K scores, Gumbel noise plus
-focus * p for orbital p.  focus = 0 draws the (alpha, beta) sector uniformly
(the benchmark's batches: samples spread out, hardly ever connected);
focus > 0 gathers them about the lowest determinant, as a trained
wavefunction's samples are, so that each is connected to many others.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2506_23809_amd as nqs
import workloads

# ---------------------------------------------------------------- the cases


def listed():
    return [
        # the smallest call: all 400 states of the 12-qubit sector, one full
        # VMC step; launches and latency are all there is
        {"name": "step-12q-400", "kind": "step", "orbitals": 6, "n": 400, "focus": 0.0,
         "precision": "fp64"},
        # an early VMC step of the 40-qubit molecule, about the 4,000 unique
        # samples per process that weak-scaling runs use
        {"name": "step-40q-4096", "kind": "step", "orbitals": 20, "n": 4096, "focus": 0.4,
         "precision": "fp64"},
        # the 40-qubit benchmark batch: uniform sector samples
        {"name": "step-40q-65536", "kind": "step", "orbitals": 20, "n": 65536, "focus": 0.0,
         "precision": "fp64"},
        # a converged 40-qubit step: the largest per-rank share of unique
        # samples reported for a molecule of this size, gathered about the
        # reference determinant
        {"name": "step-40q-37843-near", "kind": "step", "orbitals": 20, "n": 37843,
         "focus": 0.4, "precision": "fp64"},
        # the headline benchmark batch: 100 qubits, uniform sector samples
        {"name": "step-100q-262144", "kind": "step", "orbitals": 50, "n": 262144,
         "focus": 0.0, "precision": "fp64"},
        # the same molecule once the samples gather about the reference
        {"name": "step-100q-20001-near", "kind": "step", "orbitals": 50, "n": 20001,
         "focus": 0.4, "precision": "fp64"},
        # asynchronous local energies in FP32 with compensation: two-word bit
        # strings, an odd size, moderately gathered samples
        {"name": "eloc-56q-50021-fp32k", "kind": "eloc", "orbitals": 28, "n": 50021,
         "focus": 0.25, "precision": "fp32k"},
        # the integral (Slater-Condon) form of the 40-qubit molecule
        {"name": "integrals-40q-8193-near", "kind": "integrals", "orbitals": 20, "n": 8193,
         "focus": 0.4, "precision": "fp64"},
        # a Hamiltonian outside the molecular form: strings flipping up to 12
        # qubits, no spin masks
        {"name": "pauli-36q-10007", "kind": "pauli", "qubits": 36, "groups": 20000,
         "n": 10007, "precision": "fp64"},
        # a family of molecules evaluated together: ten Hamiltonians of 24 to
        # 64 qubits with uneven batches
        {"name": "batch-10-molecules", "kind": "batch", "jobs": 10, "n": 100000, "focus": 0.1,
         "precision": "fp64"},
        # a service: 24 requests of 24- to 64-qubit molecules submitted at
        # once and drained
        {"name": "serve-24-requests", "kind": "serve", "jobs": 24, "n": 20000, "focus": 0.1,
         "precision": "fp64"},
        # Eq. 1 over local energies that are already there
        {"name": "energy-262921", "kind": "energy", "n": 262921},
    ]


STEP_ORBITALS = (6, 8, 10, 13, 16, 20, 24, 28, 31, 33, 50)
FAMILY_ORBITALS = (12, 14, 16, 20, 24, 28, 32)


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("step", "step", "step", "step", "eloc", "eloc", "integrals", "pauli",
                       "batch", "serve", "energy"))
    if kind == "energy":
        return {"kind": kind, "n": _log_int(rng, 300, 262921)}
    precision = rng.choice(("fp64", "fp64", "fp32k"))
    if kind == "pauli":
        return {"kind": kind, "qubits": rng.randint(20, 60), "groups": _log_int(rng, 500, 20000),
                "n": _log_int(rng, 300, 10007), "precision": precision}
    if kind in ("batch", "serve"):
        return {"kind": kind, "jobs": rng.randint(3, 10 if kind == "batch" else 24),
                "n": _log_int(rng, 2000, 100000 if kind == "batch" else 20000),
                "focus": round(rng.choice((0.0, rng.uniform(0.0, 0.15))), 3),
                "precision": precision}
    if kind == "integrals":
        K = rng.choice((8, 13, 20))
        return {"kind": kind, "orbitals": K, "n": min(_log_int(rng, 300, 8193), _sector(K) // 2),
                "focus": round(rng.choice((0.0, rng.uniform(0.1, 0.4))), 3), "precision": "fp64"}
    K = rng.choice(STEP_ORBITALS)
    focus = round(rng.choice((0.0, rng.uniform(0.05, 0.4))), 3)
    top = min(262144 if focus == 0.0 and K >= 16 else 37843 if K <= 33 else 20001, _sector(K) // 2)
    return {"kind": kind, "orbitals": K, "n": _log_int(rng, min(300, top // 2), top),
            "focus": focus, "precision": precision}


def _sector(K):
    """States with K // 2 alpha and K - K // 2 beta electrons."""
    return math.comb(K, K // 2) * math.comb(K, K - K // 2)


# ---------------------------------------------------------------- Hamiltonians


@functools.lru_cache(maxsize=16)
def _molecule(K):
    """(h, eri, x, z, c) of the synthetic molecule with K orbitals."""
    h, eri = workloads.integrals(np.random.default_rng([7, K]), K, 6.0 if K >= 40 else 4.0)
    return (h, eri, *workloads.jw_terms(h, eri))


@functools.lru_cache(maxsize=4)
def _pauli_table(nq, groups):
    """Strings flipping 1 to 12 of nq qubits (six Z strings each, even numbers
    of Y) and a diagonal of one- and two-qubit Z strings."""
    rng = np.random.default_rng([8, nq, groups])
    flips = rng.integers(1, 13, size=groups)
    at = np.argsort(rng.random((groups, nq)), axis=1)
    bits = np.zeros((groups, nq), bool)
    for k in range(12):
        rows = flips > k
        bits[rows, at[rows, k]] = True
    x = np.repeat(bits, 6, axis=0)
    z = rng.random((6 * groups, nq)) < 0.2
    odd = (x & z).sum(axis=1) % 2 == 1
    first = x.argmax(axis=1)
    z[odd, first[odd]] ^= True
    d = np.zeros((1 + nq + nq * (nq - 1) // 2, nq), bool)
    i, j = np.triu_indices(nq, 1)
    d[np.arange(1, 1 + nq), np.arange(nq)] = True
    d[np.arange(1 + nq, d.shape[0]), i] = True
    d[np.arange(1 + nq, d.shape[0]), j] = True
    x = np.concatenate([np.zeros_like(d), x])
    z = np.concatenate([d, z])
    c = rng.normal(0.0, 0.1, size=x.shape[0])
    return workloads.pack_bits(x), workloads.pack_bits(z), c


@functools.lru_cache(maxsize=None)
def _handle(kind, *size):
    if kind == "pauli":
        return nqs.Hamiltonian(*_pauli_table(*size), size[0])
    h, eri, x, z, c = _molecule(size[0])
    if kind == "integrals":
        return nqs.Hamiltonian.from_integrals(h, eri)
    return nqs.Hamiltonian(x, z, c, 2 * size[0], workloads.spin_masks(2 * size[0]))


@functools.lru_cache(maxsize=None)
def _server(precision, largest):
    """A server of four lanes with every molecule of the family registered."""
    s = nqs.Server(32 << 30, streams=4, precision=precision)
    for K in FAMILY_ORBITALS:
        s.add(_handle("molecule", K), largest)
    return s


# ---------------------------------------------------------------- samples


def _words(idx, spin):
    """Sample words of occupied orbitals idx [m, k]: qubit 2 p + spin of orbital p."""
    q = 2 * idx + spin
    one = torch.ones_like(q)
    lo = torch.where(q < 64, one << (q & 63), 0).sum(dim=1)
    hi = torch.where(q >= 64, one << (q & 63), 0).sum(dim=1)
    return torch.stack([lo, hi], dim=1)


def _unique(words, gen):
    """The distinct rows of words [m, 2], in random order."""
    key = words[:, 0] * -7046029254386353131 + words[:, 1] * -4658895280553007687
    key, at = torch.sort(key, stable=True)
    keep = torch.ones_like(key, dtype=torch.bool)
    keep[1:] = key[1:] != key[:-1]
    words = words[at[keep]]
    return words[torch.randperm(words.shape[0], generator=gen, device=words.device)]


def _grow(n, gen, make):
    """n distinct samples of make(m) (m draws, [m, 2])."""
    words = make(2 * n)
    for _ in range(200):
        words = _unique(words, gen)
        if words.shape[0] >= n:
            return words[:n].contiguous()
        words = torch.cat([words, make(2 * n)])
    raise ValueError("too few distinct samples for this case")


def _orbital_samples(K, n, focus, gen):
    def make(m):
        out = 0
        for spin, k in ((0, K // 2), (1, K - K // 2)):
            u = torch.rand((m, K), generator=gen, device="cuda", dtype=torch.float64)
            score = -torch.log(-torch.log(u.clamp_(1e-300, 1.0 - 1e-16)))
            score -= focus * torch.arange(K, device="cuda")
            out = out + _words(score.topk(k, dim=1).indices, spin)
        return out
    return _grow(n, gen, make)


def _walk_samples(x, n, gen):
    """Strings up to four random flips of the table away from a few states."""
    flips = torch.from_numpy(x[(x != 0).any(axis=1)].view(np.int64)).cuda()

    def pick(m):
        return flips[torch.randint(flips.shape[0], (m,), generator=gen, device="cuda")]

    roots = pick(8) ^ pick(8)

    def make(m):
        w = roots[torch.randint(8, (m,), generator=gen, device="cuda")]
        for _ in range(4):
            go = torch.rand(m, generator=gen, device="cuda") < 0.5
            w = torch.where(go[:, None], w ^ pick(m), w)
        return w
    return _grow(n, gen, make)


def _amplitudes(S, focus, gen):
    """log|psi|, phase and counts of a batch: log|psi| ~ N(0, 2) for spread
    batches; for gathered ones it falls with the orbitals' heights."""
    n = S.shape[0]
    la = torch.randn(n, generator=gen, device="cuda", dtype=torch.float64)
    if focus > 0.0:
        height = torch.zeros_like(la)
        for q in range(128):
            height += ((S[:, q >> 6] >> (q & 63)) & 1) * (q // 2)
        la = 0.5 * la - 0.25 * focus * (height - height.min())
    else:
        la = 2.0 * la
    ph = torch.rand(n, generator=gen, device="cuda", dtype=torch.float64) * (2.0 * math.pi)
    w = torch.empty(n, device="cuda", dtype=torch.float64).geometric_(0.3, generator=gen)
    return la, ph, w.to(torch.int64)


def _family(case):
    """(orbitals, samples) of each job: sizes spread over a factor of a
    hundred below the case's n."""
    jobs = []
    for j in range(case["jobs"]):
        K = FAMILY_ORBITALS[(3 * j) % len(FAMILY_ORBITALS)]
        share = 100.0 ** (-((7 * j) % case["jobs"]) / case["jobs"])
        jobs.append((K, max(64, int(case["n"] * share) | 1)))
    return jobs


def _inputs(case, seed):
    """The batches of a case: (samples, log|psi|, phase, counts) each."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    kind = case["kind"]
    if kind == "pauli":
        S = _walk_samples(_pauli_table(case["qubits"], case["groups"])[0], case["n"], gen)
        return [(S, *_amplitudes(S, 0.0, gen))]
    jobs = _family(case) if kind in ("batch", "serve") else [(case["orbitals"], case["n"])]
    got = []
    for K, n in jobs:
        S = _orbital_samples(K, n, case["focus"], gen)
        got.append((S, *_amplitudes(S, case["focus"], gen)))
    return got


# ---------------------------------------------------------------- the calls


def prepare(case, seed):
    kind = case["kind"]
    if kind == "energy":
        gen = torch.Generator(device="cuda")
        gen.manual_seed(int(seed))
        n = case["n"]
        e = torch.randn((n, 2), generator=gen, device="cuda", dtype=torch.float64)
        e[:, 0] -= 100.0
        w = torch.empty(n, device="cuda", dtype=torch.float64).geometric_(0.3, generator=gen)
        return {"kind": kind, "eloc": e, "w": w.to(torch.int64)}
    state = {"kind": kind, "precision": case["precision"], "in": _inputs(case, seed)}
    state["out"] = [torch.empty((b[0].shape[0], 2), dtype=torch.float64, device="cuda")
                    for b in state["in"]]
    if kind == "pauli":
        state["ham"] = _handle(kind, case["qubits"], case["groups"])
    elif kind in ("step", "eloc"):
        state["ham"] = _handle("molecule", case["orbitals"])
    elif kind == "integrals":
        state["ham"] = _handle(kind, case["orbitals"])
    elif kind == "serve":
        state["hams"] = [_handle("molecule", K) for K, _ in _family(case)]
        state["server"] = _server(case["precision"], 20001)
        torch.cuda.current_stream().synchronize()  # the lanes have streams of their own
    else:
        # a handle appears once in a batch: every job has its own molecule
        # handle, kept by the plan
        jobs = [(nqs.Hamiltonian(*_molecule(K)[2:], 2 * K, workloads.spin_masks(2 * K)), *b, out)
                for (K, _), b, out in zip(_family(case), state["in"], state["out"])]
        state["batch"] = nqs.Batch(
            [(ham, S, la, ph, w, out) for ham, S, la, ph, w, out in jobs],
            precision=case["precision"])
    return state


def run(state):
    kind = state["kind"]
    if kind == "energy":
        mean, var, sum_w = nqs.energy(state["w"], state["eloc"])
        return {"mean": np.complex128(mean), "var": var, "sum_w": sum_w}
    if kind == "batch":
        state["batch"].launch()
        return state["out"]
    if kind == "serve":
        server = state["server"]
        for ham, b, out in zip(state["hams"], state["in"], state["out"]):
            server.submit(ham, *b, out)
        server.drain()
        server.poll()
        return state["out"]
    S, la, ph, w = state["in"][0]
    if kind == "step":
        out = state["out"][0]
        mean, var, sum_w = state["ham"].eloc_energy_into(out, S, la, ph, w,
                                                         precision=state["precision"])
        return {"eloc": out, "mean": np.complex128(mean), "var": var, "sum_w": sum_w}
    return state["ham"].eloc(S, la, ph, w, precision=state["precision"])


def work(case):
    """Per sample: bit string, log|psi|, phase, count and E_loc once, and the
    multiply-adds of the diagonal's triangle (connected pairs come on top)."""
    if case["kind"] == "energy":
        return {"bytes": 24 * case["n"], "flops": 9 * case["n"]}
    if case["kind"] == "pauli":
        jobs = [(case["qubits"], case["n"])]
    elif case["kind"] in ("batch", "serve"):
        jobs = [(2 * K, n) for K, n in _family(case)]
    else:
        jobs = [(2 * case["orbitals"], case["n"])]
    return {"bytes": sum(56 * n for _, n in jobs),
            "flops": sum(n * nq * (nq + 1) for nq, n in jobs)}


# ---------------------------------------------------------------- 64-bit values


def _popcount(v):
    v = v - ((v >> 1) & 0x5555555555555555)
    v = (v & 0x3333333333333333) + ((v >> 2) & 0x3333333333333333)
    v = (v + (v >> 4)) & 0x0F0F0F0F0F0F0F0F
    return ((v * 0x0101010101010101) >> 56) & 0x7F


class _Table:
    """Pauli terms grouped by flip mask, for lookups of many masks at once."""

    def __init__(self, nq, x, z, c):
        x = torch.from_numpy(np.ascontiguousarray(x).view(np.int64)).cuda()
        z = torch.from_numpy(np.ascontiguousarray(z).view(np.int64)).cuda()
        c = torch.from_numpy(np.ascontiguousarray(c)).cuda()
        self.nq = nq
        ny = _popcount(x[:, 0] & z[:, 0]) + _popcount(x[:, 1] & z[:, 1])
        c = torch.where((ny // 2) % 2 == 1, -c, c)
        diag = (x == 0).all(dim=1)
        # diagonal: strings of at most two Z, as s^T U s with s = 1 - 2 n
        zb = self.bits(z[diag])
        count = zb.sum(dim=1)
        assert int(count.max()) <= 2
        last = nq - 1 - zb.flip(1).to(torch.int8).argmax(dim=1)
        first = zb.to(torch.int8).argmax(dim=1)
        cd = c[diag]
        self.d0 = cd[count == 0].sum()
        self.d1 = torch.zeros(nq, dtype=torch.float64, device="cuda")
        self.d1.index_add_(0, first[count == 1], cd[count == 1])
        self.d2 = torch.zeros((nq, nq), dtype=torch.float64, device="cuda")
        self.d2[first[count == 2], last[count == 2]] = cd[count == 2]
        x, z, c = x[~diag], z[~diag], c[~diag]
        key, at = torch.sort(self.key(x), stable=True)
        self.z, self.c, x = z[at], c[at], x[at]
        self.keys, self.size = torch.unique_consecutive(key, return_counts=True)
        self.begin = torch.cumsum(self.size, 0) - self.size
        self.x = x[self.begin]
        assert bool((torch.repeat_interleave(self.x, self.size, dim=0) == x).all())
        self.flips = int((_popcount(x[:, 0]) + _popcount(x[:, 1])).max())

    @staticmethod
    def key(w):
        return w[:, 0] * -7046029254386353131 + w[:, 1] * -4658895280553007687

    def bits(self, w):
        q = torch.arange(self.nq, device="cuda")
        return ((w[:, (q >> 6)] >> (q & 63)) & 1).to(torch.bool)

    def diagonal(self, S):
        s = 1.0 - 2.0 * self.bits(S).to(torch.float64)
        return self.d0 + s @ self.d1 + ((s @ self.d2) * s).sum(dim=1)

    def element(self, S, d):
        """(which rows of d are flips of the table, <x|H|x ^ d> of those)."""
        g = torch.searchsorted(self.keys, self.key(d)).clamp_(max=self.keys.shape[0] - 1)
        ok = torch.nonzero((self.x[g] == d).all(dim=1)).flatten()
        g, S = g[ok], S[ok]
        size, t0 = self.size[g], self.begin[g]
        v = torch.zeros(g.shape[0], dtype=torch.float64, device="cuda")
        live = torch.arange(g.shape[0], device="cuda")
        for t in range(int(size.max()) if g.shape[0] else 0):
            live = live[size[live] > t]
            z, c = self.z[t0[live] + t], self.c[t0[live] + t]
            par = _popcount(z[:, 0] & S[live, 0]) + _popcount(z[:, 1] & S[live, 1])
            v.index_add_(0, live, torch.where(par % 2 == 1, -c, c))
        return ok, v


@functools.lru_cache(maxsize=2)
def _table(kind, *size):
    if kind == "pauli":
        return _Table(size[0], *_pauli_table(*size))
    return _Table(2 * size[0], *_molecule(size[0])[2:])


def _exact_eloc(tab, S, la, ph):
    """E_loc of every sample by comparing all pairs of samples."""
    n, nq = S.shape[0], tab.nq
    e = torch.zeros((n, 2), dtype=torch.float64, device="cuda")
    e[:, 0] = tab.diagonal(S)
    s = torch.where(tab.bits(S), 1.0, -1.0).to(torch.float16)
    right = s.t().contiguous()
    rows = max(1, min(n, (1 << 29) // n))
    for r in range(0, n, rows):
        # +-1 products: nq - 2 distance
        near = (s[r:r + rows] @ right) >= nq - 2 * tab.flips
        i, j = near.nonzero(as_tuple=True)
        i = i + r
        keep = i != j
        i, j = i[keep], j[keep]
        for a in range(0, i.shape[0], 1 << 23):
            ii, jj = i[a:a + (1 << 23)], j[a:a + (1 << 23)]
            ok, h = tab.element(S[ii], S[ii] ^ S[jj])
            ii, jj = ii[ok], jj[ok]
            m, f = h * torch.exp(la[jj] - la[ii]), ph[jj] - ph[ii]
            e.index_add_(0, ii, torch.stack([m * torch.cos(f), m * torch.sin(f)], dim=1))
    return e


def _exact_energy(w, e):
    w = w.to(torch.float64)
    mean = (w[:, None] * e).sum(dim=0) / w.sum()
    var = (w * ((e - mean) ** 2).sum(dim=1)).sum() / w.sum()
    return {"mean": np.complex128(complex(float(mean[0]), float(mean[1]))), "var": float(var),
            "sum_w": float(w.sum())}


def exact(case, seed):
    kind = case["kind"]
    if kind == "energy":
        state = prepare(case, seed)
        return _exact_energy(state["w"], state["eloc"])
    batches = _inputs(case, seed)
    if kind in ("batch", "serve"):
        return [_exact_eloc(_table("molecule", K), S, la, ph)
                for (K, _), (S, la, ph, _) in zip(_family(case), batches)]
    S, la, ph, w = batches[0]
    tab = (_table(kind, case["qubits"], case["groups"]) if kind == "pauli"
           else _table("molecule", case["orbitals"]))
    e = _exact_eloc(tab, S, la, ph)
    if kind == "step":
        return {"eloc": e, **_exact_energy(w, e)}
    return torch.view_as_complex(e)
