"""nqs_eloc_energy after a call that ran the pair join (it then launches the
join's kernels alone): what the device decides, and so every bit of E_loc,
depends on the batch and not on the call before, and a batch is evaluated once
unless the join is declined.

Batches: spread samples, for which the join runs, then ones gathered about the
lowest determinant but far from filling a partition, for which comparing all
pairs costs less.  Occupied orbitals are the largest of K scores, Gumbel noise
less focus * p for orbital p.
"""
import numpy as np
import pytest

import paper_2506_23809_amd as nqs
import workloads as W
from test_gpu_pairs import say

pytestmark = pytest.mark.gpu


def scored_samples(K, na, nb, n, focus, seed):
    """n distinct states of the sector."""
    rng = np.random.default_rng([seed, K, n])
    got = np.zeros((0, 2), np.uint64)
    while got.shape[0] < n:
        b = np.zeros((n, 2 * K), bool)
        for spin, k in ((0, na), (1, nb)):
            score = rng.gumbel(size=(n, K)) - focus * np.arange(K)
            top = np.argpartition(-score, k, axis=1)[:, :k]
            b[np.arange(n)[:, None], 2 * top + spin] = True
        got = np.unique(np.concatenate([got, W.pack_bits(b)]), axis=0)
    return got[rng.permutation(got.shape[0])[:n]]


def inputs(torch, S, seed):
    n = S.shape[0]
    rng = np.random.default_rng([seed, n])
    return (nqs.to_device_samples(S), torch.from_numpy(rng.normal(0.0, 1.0, n)).cuda(),
            torch.from_numpy(rng.uniform(0.0, 6.0, n)).cuda(),
            torch.from_numpy(rng.integers(1, 9, n)).cuda())


def step(torch, ham, batch):
    out = torch.full((batch[0].shape[0], 2), float("nan"), dtype=torch.float64, device="cuda")
    res = ham.eloc_energy_into(out, *batch)
    return out.cpu().numpy().view(np.uint64), res


def evaluations(torch, fn):
    """Evaluations within fn (each has one finish kernel)."""
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        fn()
        torch.cuda.synchronize()
    names = [e.name for e in prof.events()]
    if not any("finish" in v for v in names):
        pytest.skip("the profiler sees no kernels here")
    return sum("eloc_finish" in v for v in names)


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "a GPU is required"
    nqs.load_library()
    return torch


@pytest.mark.parametrize("K,n,focus", [(20, 9000, 0.15), (20, 9000, 0.2), (20, 20000, 0.15),
                                       (50, 9000, 0.1), (50, 20001, 0.05)])
def test_decision_is_the_full_launchs(torch_dev, workload_cache, K, n, focus):
    torch = torch_dev
    h, eri = W.integrals(np.random.default_rng([31, K]), K, 4.0)
    x, z, c = workload_cache(("terms", K), lambda: W.jw_terms(h, eri)[:3])
    spread = inputs(torch, scored_samples(K, K // 2, K // 2, n, 0.0, 1), 1)
    near = inputs(torch, scored_samples(K, K // 2, K // 2, n, focus, 2), 2)
    fresh = nqs.Hamiltonian(x, z, c, 2 * K, W.spin_masks(2 * K))
    ham = nqs.Hamiltonian(x, z, c, 2 * K, W.spin_masks(2 * K))
    say(f"decision: {2 * K} qubits, {n} samples, focus {focus}")
    ref = torch.view_as_real(fresh.eloc(*near)).cpu().numpy().view(np.uint64)
    fresh.sync()
    want = fresh.plan()["join_ran"]
    for _ in range(3):
        step(torch, ham, spread)
        assert ham.plan()["join_ran"] == 1
    for _ in range(3):
        got, res = step(torch, ham, near)
        assert ham.plan()["join_ran"] == want == 0
        assert np.array_equal(got, ref)
    # (the same sums from a handle that never joined)
    assert step(torch, fresh, near)[1] == res
    ham.close()
    fresh.close()


def test_a_joined_batch_is_evaluated_once(torch_dev):
    """A general table (no enumeration) whose full launch accepts the join."""
    torch = torch_dev
    rng = np.random.default_rng(17)
    nq, G, n = 36, 500, 10007
    flips = np.zeros((G, nq), bool)
    for g in range(G):
        flips[g, rng.choice(nq, int(rng.integers(1, 6)), replace=False)] = True
    zs = rng.random((G, nq)) < 0.2
    odd = (flips & zs).sum(axis=1) % 2 == 1
    zs[odd, flips.argmax(axis=1)[odd]] ^= True
    general = nqs.Hamiltonian(W.pack_bits(flips), W.pack_bits(zs), rng.normal(size=G), nq, None)
    S = np.unique(W.pack_bits(rng.random((n + 50, nq)) < 0.5), axis=0)
    batch = inputs(torch, S[rng.permutation(S.shape[0])[:n]], 3)
    step(torch, general, batch)
    say("evaluations: general table, spread samples")
    assert general.plan()["join_ran"] == 1
    assert evaluations(torch, lambda: step(torch, general, batch)) == 1
    general.close()


def test_a_batch_below_the_grouping_is_evaluated_once(torch_dev):
    """The step after a joined one that has no join to launch."""
    torch = torch_dev
    K = 20
    h, eri = W.integrals(np.random.default_rng([31, K]), K, 4.0)
    ham = nqs.Hamiltonian(*W.jw_terms(h, eri)[:3], 2 * K, W.spin_masks(2 * K))
    large = inputs(torch, scored_samples(K, 10, 10, 9000, 0.0, 1), 1)
    small = inputs(torch, scored_samples(K, 10, 10, 8192, 0.0, 4), 4)
    step(torch, ham, large)
    assert ham.plan()["join_ran"] == 1
    say("evaluations: molecule, a joined batch and then one below the grouping")
    assert evaluations(torch, lambda: step(torch, ham, large)) == 1
    assert evaluations(torch, lambda: step(torch, ham, small)) == 1
    assert ham.plan()["join_ran"] == -1
    ham.close()
