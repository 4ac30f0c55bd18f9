"""Repeated evaluations of one batch give identical bits in every strategy,
also where the order in which a sample's hits are added differs from call to
call (the pair join places the members of a group by atomics): two-word and
one-word bit strings below the matrix tiles' line, and above it."""
import numpy as np
import pytest

import paper_2506_23809_amd as nqs
import workloads as W
from test_gpu_pairs import near_samples, run, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,n", [(33, 900), (20, 1500), (12, 1200), (50, 2000)])
@pytest.mark.parametrize("precision", ["fp64", "fp32k"])
def test_repeated_calls_give_identical_bits(K, n, precision):
    import torch
    assert torch.cuda.is_available(), "a GPU is required"
    nqs.load_library()
    h, eri = W.integrals(np.random.default_rng([31, K]), K, 4.0)
    ham = nqs.Hamiltonian(*W.jw_terms(h, eri)[:3], 2 * K, W.spin_masks(2 * K))
    rng = np.random.default_rng([5, K])
    S = near_samples(K, K // 2, K // 2, n, 13)
    la, ph = rng.normal(0.0, 1.0, n), rng.uniform(0.0, 6.0, n)
    for strategy in ("join", "auto", "enum", "stream"):
        if K == 50 and strategy == "stream":
            continue  # two million groups past every sample
        say(f"repeated: {2 * K} qubits, {n} samples, {precision}, {strategy}")
        first = run(torch, ham, S, la, ph, precision, strategy)
        assert first[1]["hits"] > 10 * n
        for _ in range(6):
            e = run(torch, ham, S, la, ph, precision, strategy)[0]
            assert np.array_equal(e.view(np.uint64), first[0].view(np.uint64)), strategy
    ham.close()
