"""One VMC step of a small batch (`nqs_eloc_energy`): up to 512 samples the
finish kernel is one block and publishes the energy itself.  Sizes about the
wave and about the line; eager, captured and replayed calls; E_loc bits equal to
`nqs_eloc_eval`'s, read on another stream as soon as the call returns; the
energy within 1e-12 of the oracle's (as the larger batches' test)."""
import numpy as np
import pytest

import oracle
import paper_2506_23809_amd as nqs
import workloads as W
from test_gpu_pairs import near_samples, say

pytestmark = pytest.mark.gpu

K = 8


@pytest.mark.parametrize("n", [1, 63, 64, 65, 511, 512, 513])
@pytest.mark.parametrize("precision", ["fp64", "fp32k"])
def test_small_step(n, precision):
    import torch
    assert torch.cuda.is_available(), "a GPU is required"
    nqs.load_library()
    h, eri = W.integrals(np.random.default_rng([31, K]), K, 4.0)
    x, z, c = W.jw_terms(h, eri)[:3]
    S = nqs.to_device_samples(near_samples(K, K // 2, K // 2, n, 3))
    rng = np.random.default_rng([3, n])
    la = torch.from_numpy(rng.normal(0.0, 1.0, n)).cuda()
    ph = torch.from_numpy(rng.uniform(0.0, 6.0, n)).cuda()
    wt_np = rng.integers(0, 9, n) + (n == 1)
    wt = torch.from_numpy(wt_np).cuda()
    ham = nqs.Hamiltonian(x, z, c, 2 * K, W.spin_masks(2 * K))
    say(f"small step: n = {n}, {precision}")
    ref = torch.view_as_real(ham.eloc(S, la, ph, wt, precision=precision)).cpu().numpy()
    ham.sync()
    side = torch.cuda.Stream()
    out = torch.empty((n, 2), dtype=torch.float64, device="cuda")
    results = []
    for r in range(5):
        out.fill_(float("nan"))
        results.append(ham.eloc_energy_into(out, S, la, ph, wt, precision=precision))
        with torch.cuda.stream(side):
            got = out.cpu().numpy()
        assert np.array_equal(got.view(np.uint64), ref.view(np.uint64)), r
    assert all(res == results[0] for res in results)
    m, v, sw = results[0]
    el = ref[:, 0] + 1j * ref[:, 1]
    m_ref, v_ref, sw_ref = oracle.energy(wt_np, el)
    scale = float(np.sum(wt_np * np.abs(el)) / np.sum(wt_np))
    assert sw == sw_ref
    assert abs(m - m_ref) <= 2e-12 * scale
    assert abs(v - v_ref) <= 1e-12 * max(scale * scale, v_ref)
    bad = wt.clone()
    bad[n // 2] = -1
    with pytest.raises(nqs.NQSError) as ex:
        ham.eloc_energy_into(out, S, la, ph, bad, precision=precision)
    assert ex.value.code == nqs.NQS_E_RANGE
    ham.close()
