"""Group records: tabulated groups (strings that differ only in the flipped
qubits), occupation rows (strings that differ from a common base in one
qubit) and general groups, for one to four flips, against the CPU oracle, on
samples of every sector (both parities of the bits at the flips), in every
strategy.  Tolerances: 1e-12 A(x) in FP64, 1e-6 A(x) in FP32 with
compensation.
"""
import math
import sys

import numpy as np
import pytest

import oracle
import paper_2506_23809_amd as nqs
import workloads as W

pytestmark = pytest.mark.gpu


def _table(nq, rng):
    """Groups of one to four flips of every form, and a diagonal."""
    xs, zs = [], []
    for g in range(160):
        m = 1 + g % 4
        x = np.zeros(nq, bool)
        x[rng.choice(nq, m, replace=False)] = True
        at = np.nonzero(x)[0]
        base = rng.random(nq) < 0.4
        base[at] = False
        form = (g // 4) % 4
        if form == 0:      # one string
            outs = [base]
        elif form == 1:    # one base, every even subset of the flips
            outs = [base] * 8
        elif form == 2:    # base and single qubits: an occupation row for m <= 2
            outs = [base]
            for r in rng.permutation(np.nonzero(~x)[0])[:nq - 5]:
                o = base.copy()
                o[r] ^= True
                outs.append(o)
        else:              # unrelated strings
            outs = [(rng.random(nq) < 0.4) & ~x for _ in range(int(rng.integers(2, 14)))]
        for k, o in enumerate(outs):
            z = o.copy()
            flip = [int(rng.integers(0, 2)) for _ in at] if form != 1 else [(k >> i) & 1 for i in range(m)]
            if sum(flip) % 2:
                flip[0] ^= 1
            z[at] = np.array(flip, bool)
            xs.append(x)
            zs.append(z)
    for _ in range(40):    # a diagonal with strings of any length
        xs.append(np.zeros(nq, bool))
        zs.append(rng.random(nq) < 0.2)
    return W.pack_bits(np.array(xs)), W.pack_bits(np.array(zs))


@pytest.mark.parametrize("nq", [24, 63, 64, 90])
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32k", 1e-6)])
def test_group_forms_agree_with_the_oracle(nq, precision, tol):
    import torch
    assert torch.cuda.is_available(), "a GPU is required"
    rng = np.random.default_rng([41, nq])
    x, z = _table(nq, rng)
    c = rng.normal(size=x.shape[0])
    moves = x[(x != 0).any(axis=1)]
    roots = W.pack_bits(rng.random((6, nq)) < 0.5)
    S = roots[rng.integers(0, 6, 900)]
    for _ in range(2):
        S = np.where(rng.random(900)[:, None] < 0.7, S ^ moves[rng.integers(0, len(moves), 900)], S)
    S = np.unique(np.concatenate([roots, S]), axis=0)
    S = S[rng.permutation(S.shape[0])]
    n = S.shape[0]
    la, ph = rng.normal(0, 1, n), rng.uniform(0, 2 * math.pi, n)
    ref, ab, nc = oracle.eloc(nq, x, z, c, S, la, ph)
    ham = nqs.Hamiltonian(x, z, c, nq, None)
    St = nqs.to_device_samples(S)
    la_t, ph_t = torch.from_numpy(la).cuda(), torch.from_numpy(ph).cuda()
    for strategy in ("auto", "stream", "join"):
        print(f"[gpu-groups] {nq} qubits, {n} samples, {precision}, {strategy}", flush=True)
        sys.stdout.flush()
        ham.set_tuning(strategy=strategy)
        e = ham.eloc(St, la_t, ph_t, precision=precision)
        ham.sync()
        got = e.cpu().numpy()
        assert np.all(np.abs(got - ref) <= tol * ab), strategy
        assert ham.stats()["hits"] == int(nc.sum()) - n > 500
    ham.close()
