"""The comparison of all pairs of samples on the matrix cores (what AUTO runs
for small batches, and beside the pair join for gathered ones) against the
CPU oracle and against the other strategies, through the C ABI.

Floating point within 1e-12 A(x) (FP64) or 1e-6 A(x) (FP32 with
compensation) of the oracle; hit counts equal the oracle's connected pairs;
debug dumps equal the streaming kernel's.  Sizes sit at the edges of the
32-sample tiles, of the one- and two-word bit strings, of the two column
shares and of the batch size from which samples are grouped first.
"""
import math
import sys

import numpy as np
import pytest

import oracle
import paper_2506_23809_amd as nqs
import workloads as W

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32k": 1e-6}


def say(msg):
    print(f"[gpu-pairs] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "a GPU is required"
    nqs.load_library()
    return torch


def near_samples(K, na, nb, n, seed):
    """n unique states of the sector about its lowest determinant: a few
    random exchanges of occupied and virtual orbitals each."""
    rng = np.random.default_rng([seed, K, n])
    seen, out = set(), []
    base = np.zeros(2 * K, bool)
    base[0:2 * na:2] = True
    base[1:2 * nb:2] = True
    while len(out) < n:
        b = base.copy()
        for _ in range(int(rng.integers(0, 4)) + (2 if len(out) > n // 2 else 0)):
            s = int(rng.integers(0, 2))
            o = np.nonzero(b[s::2])[0]
            v = np.nonzero(~b[s::2])[0]
            b[2 * rng.choice(o) + s] = False
            b[2 * rng.choice(v) + s] = True
        key = b.tobytes()
        if key not in seen:
            seen.add(key)
            out.append(b)
    return W.pack_bits(np.array(out))[rng.permutation(n)]


def run(torch, ham, S, la, ph, precision="fp64", strategy="auto"):
    ham.set_tuning(strategy=strategy)
    e = torch.view_as_real(ham.eloc(nqs.to_device_samples(S), torch.from_numpy(la).cuda(),
                                    torch.from_numpy(ph).cuda(), precision=precision))
    ham.sync()
    r = e.cpu().numpy()
    return np.ascontiguousarray(r).view(np.complex128)[:, 0], ham.stats(), ham.plan()


@pytest.fixture(scope="module")
def tables():
    made = {}

    def get(K):
        if K not in made:
            h, eri = W.integrals(np.random.default_rng([31, K]), K, 4.0)
            made[K] = (h, eri) + tuple(W.jw_terms(h, eri))
        return made[K]
    return get


# (orbitals, alpha, beta, samples): one tile and its edges, 62, 64 and 66
# qubits, one share and two, just below and above the grouping's 8,192
SHAPES = [(6, 3, 3, 1), (6, 3, 3, 31), (6, 3, 3, 32), (6, 3, 3, 33), (6, 2, 4, 225),
          (31, 4, 5, 97), (32, 5, 4, 640), (33, 6, 6, 1025), (12, 6, 5, 8192), (12, 6, 6, 8193),
          (16, 8, 8, 16390)]


@pytest.mark.parametrize("K,na,nb,n", SHAPES)
@pytest.mark.parametrize("precision", ["fp64", "fp32k"])
def test_pairs_agree_with_the_oracle(torch_dev, tables, K, na, nb, n, precision):
    _, _, x, z, c = tables(K)
    if n <= 400:
        S = W.sector_states(K, na, nb)[:n] if K == 6 else near_samples(K, na, nb, n, 1)
    else:
        S = near_samples(K, na, nb, n, 1)
    rng = np.random.default_rng([2, K, n])
    la, ph = rng.normal(0, 1, n), rng.uniform(0, 2 * math.pi, n)
    ham = nqs.Hamiltonian(x, z, c, 2 * K, W.spin_masks(2 * K))
    say(f"{2 * K} qubits, {n} samples, {precision}")
    e, st, plan = run(torch_dev, ham, S, la, ph, precision)
    # neither the enumeration nor the join ran: all ordered pairs were tested
    assert st["enum_rounds"] == 0 and plan["join_ran"] == (-1 if n <= 8192 else 0)
    assert st["candidates"] == n * (n - 1)
    ref, ab, nc = oracle.eloc(2 * K, x, z, c, S, la, ph)
    assert np.all(np.abs(e - ref) <= TOL[precision] * ab)
    assert st["hits"] == int(nc.sum()) - n
    ham.close()


@pytest.mark.parametrize("K,n", [(6, 400), (20, 900), (33, 500)])
def test_pairs_dumps_equal_streaming(torch_dev, tables, K, n):
    torch = torch_dev
    _, _, x, z, c = tables(K)
    S = W.sector_states(6, 3, 3) if K == 6 else near_samples(K, 4, 4, n, 3)
    rng = np.random.default_rng([4, K])
    la = torch.from_numpy(rng.normal(0, 1, n)).cuda()
    ph = torch.from_numpy(rng.uniform(0, 2 * math.pi, n)).cuda()
    ham = nqs.Hamiltonian(x, z, c, 2 * K, W.spin_masks(2 * K))
    G, T, _ = ham.info()
    got = {}
    for strategy in ("auto", "stream"):
        say(f"{2 * K} qubits, {n} samples: dump, {strategy}")
        ham.set_tuning(strategy=strategy)
        hit = torch.full((n, G), -7, dtype=torch.int32, device="cuda")
        bits = torch.zeros((n, (T + 31) // 32), dtype=torch.int32, device="cuda")
        ham.debug_dump(nqs.to_device_samples(S), la, ph, hit, bits)
        ham.sync()
        got[strategy] = (hit.cpu().numpy(), bits.cpu().numpy())
    assert np.array_equal(got["auto"][0], got["stream"][0])
    assert np.array_equal(got["auto"][1], got["stream"][1])
    assert (got["auto"][0] >= 0).sum() > n
    ham.close()


def test_pairs_integral_form_mixed_sectors_and_errors(torch_dev, tables):
    """The Slater-Condon form equals the Pauli form's oracle; samples of two
    sectors; a duplicate, a bit beyond the register and a negative count are
    latched; an infinite amplitude ratio stays infinite."""
    torch = torch_dev
    h, eri, x, z, c = tables(12)
    n = 700
    S = np.concatenate([near_samples(12, 6, 5, n // 2, 5), near_samples(12, 5, 6, n // 2, 6)])
    rng = np.random.default_rng(7)
    la, ph = rng.normal(0, 1, n), rng.uniform(0, 2 * math.pi, n)
    ref, ab, nc = oracle.eloc(24, x, z, c, S, la, ph)
    for ham in (nqs.Hamiltonian(x, z, c, 24, W.spin_masks(24)),
                nqs.Hamiltonian.from_integrals(h, eri)):
        say("mixed sectors")
        e, st, _ = run(torch, ham, S, la, ph)
        assert st["candidates"] == n * (n - 1)
        assert np.all(np.abs(e - ref) <= 1e-12 * ab)
        for what, code in (("duplicate", nqs.NQS_E_DUPLICATE), ("bit", nqs.NQS_E_RANGE),
                           ("count", nqs.NQS_E_RANGE)):
            say(f"error: {what}")
            bad = S.copy()
            w = torch.ones(n, dtype=torch.int64, device="cuda")
            if what == "duplicate":
                bad[17] = bad[600]
            elif what == "bit":
                bad[5, 0] |= np.uint64(1 << 30)
            else:
                w[9] = -1
            ham.eloc(nqs.to_device_samples(bad), torch.from_numpy(la).cuda(),
                     torch.from_numpy(ph).cuda(), w)
            with pytest.raises(nqs.NQSError) as ex:
                ham.sync()
            assert ex.value.code == code
        ham.close()
    say("an amplitude ratio that overflows")
    ham = nqs.Hamiltonian(x, z, c, 24, W.spin_masks(24))
    la2 = la.copy()
    la2[:3] = 800.0
    a, _, _ = run(torch, ham, S, la2, np.zeros(n))
    b, _, _ = run(torch, ham, S, la2, np.zeros(n), strategy="stream")
    inf_a, inf_b = np.isinf(a.real), np.isinf(b.real)
    assert inf_b.any() and np.array_equal(inf_a, inf_b)
    assert np.array_equal(np.sign(a.real[inf_a]), np.sign(b.real[inf_a]))
    ham.close()


@pytest.mark.parametrize("nq", [20, 36, 70])
def test_pairs_general_tables(torch_dev, nq):
    """Strings flipping up to 9 qubits (no pair join: more blocks than it
    takes), no spin masks."""
    rng = np.random.default_rng([9, nq])
    T = 6000
    xb = np.zeros((T, nq), bool)
    for t in range(T):
        xb[t, rng.choice(nq, rng.integers(0, 10), replace=False)] = True
    zb = rng.random((T, nq)) < 0.3
    for t in range(T):
        if np.sum(xb[t] & zb[t]) % 2:
            zb[t, np.nonzero(xb[t] & zb[t])[0][0]] = False
    x, z, c = W.pack_bits(xb), W.pack_bits(zb), rng.normal(size=T)
    base = W.pack_bits(rng.random((40, nq)) < 0.5)
    S = np.unique(np.concatenate([base, np.repeat(base, 30, axis=0) ^ x[rng.integers(0, T, 1200)]]),
                  axis=0)
    S = S[rng.permutation(S.shape[0])]
    n = S.shape[0]
    la, ph = rng.normal(0, 1, n), rng.uniform(0, 2 * math.pi, n)
    ham = nqs.Hamiltonian(x, z, c, nq, None)
    say(f"general table, {nq} qubits, {n} samples")
    e, st, plan = run(torch_dev, ham, S, la, ph)
    ref, ab, nc = oracle.eloc(nq, x, z, c, S, la, ph)
    assert plan["join_blocks"] == 0 and plan["join_ran"] == -1
    assert np.all(np.abs(e - ref) <= 1e-12 * ab)
    has_diag = bool(np.any((x[:, 0] == 0) & (x[:, 1] == 0)))
    assert st["hits"] == int(nc.sum()) - (n if has_diag else 0) > 1000
    ham.close()
