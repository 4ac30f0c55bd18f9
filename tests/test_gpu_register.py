"""Batches that hold samples with bits at or above n_qubits, in every
strategy: NQS_E_RANGE, whatever the stray bits, and the handle goes on with
the next batch as if nothing had been.  The samples share, lack or differ in
stray bits and lie among connected ones, so that pairs of them are compared
(that no table is left is shown on the CPU)."""
import numpy as np
import pytest

import paper_2506_23809_amd as nqs
import workloads as W
from test_gpu_pairs import near_samples, run, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["pauli", "integrals"])
@pytest.mark.parametrize("K,n", [(6, 300), (12, 1200), (33, 900)])
def test_stray_bits_are_an_error_and_nothing_else(K, n, form):
    import torch
    assert torch.cuda.is_available(), "a GPU is required"
    nqs.load_library()
    h, eri = W.integrals(np.random.default_rng([31, K]), K, 4.0)
    if form == "pauli":
        ham = nqs.Hamiltonian(*W.jw_terms(h, eri)[:3], 2 * K, W.spin_masks(2 * K))
    else:
        ham = nqs.Hamiltonian.from_integrals(h, eri)
    rng = np.random.default_rng([5, K])
    S = near_samples(K, K // 2, K // 2, n, 13)
    la, ph = rng.normal(0.0, 1.0, n), rng.uniform(0.0, 6.0, n)
    at = 2 * K - (64 if K > 31 else 0)  # the register ends in this word
    word = 1 if K > 31 else 0
    stray = rng.integers(0, 1 << 62, n, dtype=np.uint64) << np.uint64(at)
    stray[::3] = np.uint64(1 << 63)   # the same bit
    stray[1::3] = 0                   # none
    bad = S.copy()
    bad[:, word] |= stray
    for strategy in ("auto", "join", "stream"):
        say(f"stray bits: {form}, {2 * K} qubits, {n} samples, {strategy}")
        good = run(torch, ham, S, la, ph, strategy=strategy)[0]
        ham.eloc(nqs.to_device_samples(bad), torch.from_numpy(la).cuda(),
                 torch.from_numpy(ph).cuda())
        with pytest.raises(nqs.NQSError) as ex:
            ham.sync()
        assert ex.value.code == nqs.NQS_E_RANGE
        again = run(torch, ham, S, la, ph, strategy=strategy)[0]
        assert np.array_equal(again.view(np.uint64), good.view(np.uint64))
    ham.close()
