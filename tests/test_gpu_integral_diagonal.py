"""The integral form's diagonal: a sum over the sample's occupied orbitals,
as close as a sum in FP64 whatever the empty ones hold.

Each value is within m 2^-53 sum |t| of the exact sum of the sample's m terms
t (h_ii, the Coulomb integrals, minus the exchange ones; the bound of an FP64
sum in any order), where an unoccupied orbital has a one-electron integral of
1 to 10^8, or all integrals lie on one grid.  Single samples (whose local energy is
the diagonal alone), batches on both block sizes of the finish kernel, and a
batch plan.
"""
from fractions import Fraction

import numpy as np
import pytest

import paper_2506_23809_amd as nqs
import workloads as W
from test_gpu_pairs import say

pytestmark = pytest.mark.gpu


def terms(h, eri, occ):
    """The terms of one sample's diagonal (occ: spin orbitals 2 p + spin)."""
    t = []
    for k, i in enumerate(occ):
        a = i >> 1
        t.append(h[a, a])
        for j in occ[k + 1:]:
            b = j >> 1
            t.append(eri[a, a, b, b])
            if (i & 1) == (j & 1):
                t.append(-eri[a, b, b, a])
    return [float(v) for v in t]


def check(values, samples, h, eri, nq):
    for e, row in zip(values, W.unpack_bits(samples, nq)):
        t = terms(h, eri, np.nonzero(row)[0].tolist())
        exact = sum((Fraction(v) for v in t), Fraction(0))
        bound = len(t) * 2.0 ** -53 * sum(abs(v) for v in t)
        assert abs(Fraction(float(e.real)) - exact) <= Fraction(bound), (e, float(exact))
        assert e.imag == 0.0


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "a GPU is required"
    nqs.load_library()
    return torch


@pytest.mark.parametrize("K", [8, 33])
@pytest.mark.parametrize("large", [1.0, 1e3, 1e6, 1e8, "grid"])
def test_diagonal_of_the_integral_form(torch_dev, K, large):
    torch = torch_dev
    h, eri = W.integrals(np.random.default_rng([31, K]), K, 4.0)
    if large == "grid":
        h, eri = np.round(h * 64) / 64, np.round(eri * 1024) / 1024
        h[range(K), range(K)] = 0.0
    else:
        h[K - 1, K - 1] = large
    ham = nqs.Hamiltonian.from_integrals(h, eri)
    rng = np.random.default_rng([3, K])
    # orbital K - 1 empty but for every eighth sample; one to seven electrons
    rows = np.zeros((24, 2 * K), bool)
    for k in range(24):
        top = 2 * K if k % 8 == 0 else 2 * K - 2
        rows[k, rng.choice(top, 1 + k % 7, replace=False)] = True
    S = W.pack_bits(rows)
    say(f"integral diagonal: {2 * K} qubits, empty orbital {large}, single samples")
    zero = torch.zeros(1, dtype=torch.float64, device="cuda")
    got = []
    for k in range(24):
        e = ham.eloc(nqs.to_device_samples(S[k:k + 1]), zero, zero)
        ham.sync()
        got.append(complex(e.cpu().numpy()[0]))
    check(got, S, h, eri, 2 * K)
    say(f"integral diagonal: {2 * K} qubits, empty orbital {large}, a batch plan")
    out = torch.empty((24, 2), dtype=torch.float64, device="cuda")
    jobs = [(ham, nqs.to_device_samples(S[5:6]), zero, zero, None, out[:1])]
    b = nqs.Batch(jobs)
    b.launch()
    ham.sync()
    check([complex(*out[0].tolist())], S[5:6], h, eri, 2 * K)
    b.close()
    ham.close()


@pytest.mark.parametrize("n", [600, 262145])
def test_large_empty_orbital_in_a_batch(torch_dev, n):
    """Samples that differ pairwise in more than two electrons (no hits): the
    diagonals of a batch, on 256- and 1024-thread blocks."""
    torch = torch_dev
    K = 20
    h, eri = W.integrals(np.random.default_rng([31, K]), K, 4.0)
    h[K - 1, K - 1] = 1e8
    ham = nqs.Hamiltonian.from_integrals(h, eri)
    # distance at least six: the orbitals in triples, occupied alike
    code = np.random.default_rng(5).permutation(1 << 12)[:600]
    rows = np.zeros((code.size, 2 * K), bool)
    for k in range(12):
        for r in range(3):
            rows[:, 3 * k + r] = (code >> k) & 1
    S = W.pack_bits(rows)
    if n > S.shape[0]:
        # the rest: states with the large orbital, of amplitude zero (a few
        # are connected with the ones above)
        rng = np.random.default_rng(6)
        more = rng.integers(0, 1 << 36, 2 * n, dtype=np.uint64) | np.uint64(0x8 << 36)
        more = np.unique(more)
        more = more[rng.permutation(more.size)[:n - S.shape[0]]]
        S2 = np.concatenate([S, np.stack([more, np.zeros_like(more)], axis=1)])
    else:
        S2 = S
    la = torch.zeros(S2.shape[0], dtype=torch.float64, device="cuda")
    la[S.shape[0]:] = -float("inf")
    ph = torch.zeros_like(la)
    say(f"integral diagonal: {S2.shape[0]} samples")
    e = ham.eloc(nqs.to_device_samples(S2), la, ph)
    ham.sync()
    got = e.cpu().numpy()[:S.shape[0]]
    at = np.arange(S.shape[0])[::7]
    check([complex(got[k]) for k in at], S[at], h, eri, 2 * K)
    ham.close()
