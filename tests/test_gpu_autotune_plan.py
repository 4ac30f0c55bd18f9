"""A tuning taken from the cache is the one that was timed: an AUTO entry
stands for the built-in plan (whose filter takes 32 bits a sample where a batch
outgrows one bitmap, not the 16 that the file spells out), a forced strategy
for its own parameters."""
import numpy as np
import pytest

import paper_2506_23809_amd as nqs
import workloads as W
from test_gpu_join_only import inputs, scored_samples
from test_gpu_pairs import say

pytestmark = pytest.mark.gpu


def test_cached_tuning_is_the_timed_plan(tmp_path):
    import torch
    assert torch.cuda.is_available(), "a GPU is required"
    nqs.load_library()
    K, n = 13, 100001
    h, eri = W.integrals(np.random.default_rng([31, K]), K, 4.0)
    ham = nqs.Hamiltonian(*W.jw_terms(h, eri)[:3], 2 * K, W.spin_masks(2 * K))
    S, la, ph, _ = inputs(torch, scored_samples(K, 6, 6, n, 0.0, 41), 41)
    out = torch.empty((n, 2), dtype=torch.float64, device="cuda")
    cache = tmp_path / "tuning.json"
    say("autotune, then AUTO and a forced strategy from the cache")
    ham.autotune(S, la, ph, out, cache_path=cache)
    key = cache.read_text().split('"')[1]
    entry = '{\n  "%s": {"threads": 1024, "filter_bits": %d, "blocks_per_cu": 4, "strategy": %d, "ms": 0.1}\n}\n'

    def plan():
        ham.eloc_into(out, S, la, ph)
        ham.sync()
        return ham.plan()

    ham.set_tuning()
    built_in = plan()
    cache.write_text(entry % (key, 16, 0))
    tuning, ms = ham.autotune(S, la, ph, out, cache_path=cache)
    assert ms == -1.0 and tuning["strategy"] == "auto"
    assert plan() == built_in and built_in["filter_partitions"] == 4
    cache.write_text(entry % (key, 8, 2))
    tuning, ms = ham.autotune(S, la, ph, out, cache_path=cache)
    assert ms == -1.0 and tuning["strategy"] == "enum" and tuning["filter_bits"] == 8
    assert plan()["filter_partitions"] == 1
    ham.close()
