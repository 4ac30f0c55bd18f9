"""The pair join's matrix tiles (groups of 8 and more samples per content of
the shortest block, one-word bit strings) against the CPU oracle: sizes about
the rule's line, the 64-row waves and the 32-column steps, group sizes from a
few samples to whole batches.

Floating point within 1e-12 A(x) (FP64) or 1e-6 A(x) (FP32 with
compensation); hit counts equal the oracle's connected pairs; a candidate is an
ordered pair of a group, on either side of the line.
"""
import math

import numpy as np
import pytest

import oracle
import paper_2506_23809_amd as nqs
import workloads as W
from test_gpu_pairs import TOL, near_samples, run, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "a GPU is required"
    nqs.load_library()
    return torch


# 16 qubits: blocks of 3 and 4 qubits (the line is at 64 samples); 40: 8 (2,048)
@pytest.mark.parametrize("K,n", [(8, 63), (8, 64), (8, 65), (8, 129), (8, 1001), (20, 2047),
                                 (20, 2048), (20, 4097)])
@pytest.mark.parametrize("precision", ["fp64", "fp32k"])
def test_tiles_agree_with_the_oracle(torch_dev, workload_cache, K, n, precision):
    h, eri = W.integrals(np.random.default_rng([31, K]), K, 4.0)
    x, z, c = W.jw_terms(h, eri)[:3]
    S = near_samples(K, K // 2, K // 2, n, 7)
    rng = np.random.default_rng([7, K, n])
    la, ph = rng.normal(0.0, 2.0, n), rng.uniform(0.0, 2 * math.pi, n)
    ref, ab, nc = workload_cache(("tiles", K, n), lambda: oracle.eloc(2 * K, x, z, c, S, la, ph))
    ham = nqs.Hamiltonian(x, z, c, 2 * K, W.spin_masks(2 * K))
    say(f"tiles {2 * K} qubits, {n} samples, {precision}")
    e, st, plan = run(torch_dev, ham, S, la, ph, precision, "join")
    assert plan["join_ran"] == 1
    assert st["hits"] == int(nc.sum()) - n
    assert st["hits"] <= st["probes"] <= n * (n - 1)
    assert (np.abs(e - ref) <= TOL[precision] * ab).all()
    ham.close()


def test_tiles_latch_duplicates(torch_dev):
    K, n = 8, 300
    h, eri = W.integrals(np.random.default_rng([31, K]), K, 4.0)
    x, z, c = W.jw_terms(h, eri)[:3]
    S = near_samples(K, K // 2, K // 2, n, 7)
    S[211] = S[40]
    ham = nqs.Hamiltonian(x, z, c, 2 * K, W.spin_masks(2 * K))
    say("tiles: duplicate sample latched")
    with pytest.raises(nqs.NQSError) as ex:
        run(torch_dev, ham, S, np.zeros(n), np.zeros(n), "fp64", "join")
    assert ex.value.code == nqs.NQS_E_DUPLICATE
    ham.close()
