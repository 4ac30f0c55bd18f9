"""The comparison of all pairs in its 64-row form (batches above 32,768
samples) against the CPU oracle, and beside the pair join inside a batch plan
and in a server's lanes against single calls.

Floating point within 1e-12 A(x) (FP64) or 1e-6 A(x) (FP32 with compensation)
of the oracle, on rows at every place of the 64-row blocks and at the ragged
end; hit counts equal the streaming kernel's; batches and served requests
equal single calls bit for bit.
"""
import numpy as np
import pytest

import oracle
import paper_2506_23809_amd as nqs
import workloads as W
from test_gpu_join_only import inputs, scored_samples
from test_gpu_pairs import TOL, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "a GPU is required"
    nqs.load_library()
    return torch


def molecule(cache, K):
    def make():
        h, eri = W.integrals(np.random.default_rng([31, K]), K, 4.0)
        return (h, eri) + tuple(W.jw_terms(h, eri)[:3])
    return cache(("molecule", K), make)


def evaluate(torch, ham, batch, precision="fp64", strategy="auto"):
    ham.set_tuning(strategy=strategy)
    e = torch.view_as_real(ham.eloc(*batch, precision=precision))
    ham.sync()
    return e.cpu().numpy(), ham.stats(), ham.plan()


@pytest.mark.parametrize("K,n", [(20, 32769), (20, 32801), (33, 32769), (33, 32801)])
def test_wide_blocks_agree_with_the_oracle(torch_dev, workload_cache, K, n):
    torch = torch_dev
    h, eri, x, z, c = molecule(workload_cache, K)
    S = scored_samples(K, K // 2, K // 2, n, 0.4, 21)
    batch = inputs(torch, S, 21)
    la, ph = batch[1].cpu().numpy(), batch[2].cpu().numpy()
    rng = np.random.default_rng(22)
    rows = np.unique(np.concatenate([np.arange(64), np.arange(n - 70, n), rng.integers(0, n, 150)]))
    ref, ab, _ = oracle.eloc_rows(2 * K, x, z, c, S, la, ph, rows)
    ham = nqs.Hamiltonian(x, z, c, 2 * K, W.spin_masks(2 * K))
    say(f"wide: {2 * K} qubits, {n} samples, streaming for the hits")
    hits = evaluate(torch, ham, batch, strategy="stream")[1]["hits"]
    for precision in ("fp64", "fp32k"):
        say(f"wide: {2 * K} qubits, {n} samples, {precision}")
        e, st, plan = evaluate(torch, ham, batch, precision)
        assert st["candidates"] == n * (n - 1) and plan["join_ran"] == 0
        assert st["hits"] == hits > 10 * n
        e = e[rows, 0] + 1j * e[rows, 1]
        assert np.all(np.abs(e - ref) <= TOL[precision] * ab)
    ham.close()
    ham = nqs.Hamiltonian.from_integrals(h, eri)
    say(f"wide: {2 * K} qubits, {n} samples, integrals")
    e, st, plan = evaluate(torch, ham, batch)
    assert st["candidates"] == n * (n - 1) and st["hits"] >= hits
    e = e[rows, 0] + 1j * e[rows, 1]
    assert np.all(np.abs(e - ref) <= TOL["fp64"] * ab)
    ham.close()


# (orbitals, samples, focus, integral form): declined joins, one that runs, a
# batch below the grouping, one of 64-row blocks
JOBS = [(20, 9001, 0.3, False), (20, 9001, 0.0, False), (12, 700, 0.2, False),
        (16, 8193, 0.3, True), (33, 9000, 0.3, False), (13, 33001, 0.2, False)]


@pytest.mark.parametrize("precision", ["fp64", "fp32k"])
def test_batches_and_served_requests_equal_single_calls(torch_dev, workload_cache, precision):
    torch = torch_dev
    jobs, ref = [], []
    for k, (K, n, focus, integrals) in enumerate(JOBS):
        h, eri, x, z, c = molecule(workload_cache, K)
        ham = (nqs.Hamiltonian.from_integrals(h, eri) if integrals
               else nqs.Hamiltonian(x, z, c, 2 * K, W.spin_masks(2 * K)))
        batch = inputs(torch, scored_samples(K, K // 2, K // 2, n, focus, 30 + k), 30 + k)
        say(f"single: {2 * K} qubits, {n} samples, {precision}")
        e, st, plan = evaluate(torch, ham, batch, "fp64" if integrals else precision)
        assert plan["join_ran"] == (-1 if n <= 8192 else 1 if focus == 0.0 else 0)
        ref.append(e.view(np.uint64))
        out = torch.full((n, 2), float("nan"), dtype=torch.float64, device="cuda")
        jobs.append((ham, *batch, out))

    def equal(what):
        torch.cuda.synchronize()
        for k, (job, want) in enumerate(zip(jobs, ref)):
            assert np.array_equal(job[-1].cpu().numpy().view(np.uint64), want), (what, JOBS[k])
            job[-1].fill_(float("nan"))
        torch.cuda.synchronize()

    say("batch, launched")
    b = nqs.Batch(jobs, precision=precision)
    b.launch()
    equal("launch")
    say("batch, captured and replayed")
    s = torch.cuda.Stream()
    b.capture(s)
    for _ in range(3):
        b.replay(s)
        equal("replay")
    b.close()
    say("served")
    server = nqs.Server(8 << 30, streams=2, precision=precision)
    for job in jobs:
        server.add(job[0], 40000)
    for job in jobs:
        server.submit(*job)
    server.drain()
    done = server.poll()
    assert len(done) == len(jobs)
    equal("served")
    server.close()
    for job in jobs:
        job[0].close()
