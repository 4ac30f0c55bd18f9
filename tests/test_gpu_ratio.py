"""The FP64 amplitude ratio, formed from the two samples' amplitudes within
|log-amplitude| < 300 and from the differences outside, in every strategy.

A ratio depends on differences only, so a common offset on either side of
the line (or one that puts samples on both sides) leaves the oracle's local
energies, within 1e-12 A(x).  An amplitude of zero contributes nothing to the
other samples, and a phase that is not a number spoils every sample it reaches.
"""
import math

import numpy as np
import pytest

import oracle
import paper_2506_23809_amd as nqs
import workloads as W
from test_gpu_pairs import TOL, near_samples, run, say

pytestmark = pytest.mark.gpu

K, N = 8, 700


@pytest.fixture(scope="module")
def problem():
    import torch
    assert torch.cuda.is_available(), "a GPU is required"
    nqs.load_library()
    h, eri = W.integrals(np.random.default_rng([31, K]), K, 4.0)
    x, z, c = W.jw_terms(h, eri)[:3]
    S = near_samples(K, K // 2, K // 2, N, 11)
    rng = np.random.default_rng([11, K])
    la, ph = rng.normal(0.0, 2.0, N), rng.uniform(-9.0, 2 * math.pi, N)
    ham = nqs.Hamiltonian(x, z, c, 2 * K, W.spin_masks(2 * K))
    yield torch, ham, (x, z, c), S, la, ph
    ham.close()


@pytest.mark.parametrize("strategy", ["auto", "join", "enum", "stream"])
@pytest.mark.parametrize("offset", [0.0, -297.0, 299.5, -300.0, 1000.0, -70000.0])
def test_offsets(problem, strategy, offset):
    torch, ham, (x, z, c), S, la, ph = problem
    ref, ab, _ = oracle.eloc(2 * K, x, z, c, S, la + offset, ph)
    say(f"ratio: offset {offset}, {strategy}")
    e, _, _ = run(torch, ham, S, la + offset, ph, strategy=strategy)
    assert (np.abs(e - ref) <= TOL["fp64"] * ab).all()


@pytest.mark.parametrize("strategy", ["auto", "join", "enum", "stream"])
def test_zero_amplitude_and_nan_phase(problem, strategy):
    torch, ham, (x, z, c), S, la, ph = problem
    keep = np.arange(N) != 5
    ref, ab, _ = oracle.eloc(2 * K, x, z, c, S[keep], la[keep], ph[keep])
    la2 = la.copy()
    la2[5] = -np.inf
    say(f"ratio: a zero amplitude, {strategy}")
    e, _, _ = run(torch, ham, S, la2, ph, strategy=strategy)
    assert (np.abs(e[keep] - ref) <= TOL["fp64"] * ab).all()
    assert not np.isfinite(e[5])
    _, _, nc = oracle.eloc(2 * K, x, z, c, S, la, ph)
    alone, _, nc1 = oracle.eloc(2 * K, x, z, c, S[keep], la[keep], ph[keep])
    reached = nc[keep] > nc1  # the samples connected with sample 5
    ph2 = ph.copy()
    ph2[5] = np.nan
    say(f"ratio: a phase that is not a number, {strategy}")
    e, _, _ = run(torch, ham, S, la, ph2, strategy=strategy)
    assert reached.any() and np.array_equal(np.isnan(e[keep].real), reached)
    assert (np.abs(e[keep] - alone)[~reached] <= TOL["fp64"] * ab[~reached]).all()


@pytest.mark.parametrize("strategy", ["auto", "join", "enum", "stream"])
def test_equal_amplitudes_and_phases_leave_no_trace(problem, strategy):
    """Where all samples have one log-amplitude and one phase, every ratio is
    exactly 1: the bits of an amplitude of 1, and no imaginary part.  With one
    phase and different log-amplitudes there is none either."""
    torch, ham, _, S, la, _ = problem
    say(f"ratio: equal amplitudes and phases, {strategy}")
    zero = np.zeros(N)
    one, _, _ = run(torch, ham, S, zero, zero, strategy=strategy)
    for amp, phase in ((-7.3, 0.0), (0.1, 0.7), (-280.0, 2.9), (500.0, -1.3)):
        e, _, _ = run(torch, ham, S, zero + amp, zero + phase, strategy=strategy)
        assert np.array_equal(e.view(np.uint64), one.view(np.uint64))
    for phase in (0.7, math.pi):
        e, _, _ = run(torch, ham, S, la, zero + phase, strategy=strategy)
        assert (e.imag == 0.0).all()
