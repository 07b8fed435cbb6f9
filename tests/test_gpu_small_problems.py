"""The small problems between 17 and 64 (thin SVD by the work-group Jacobi,
CholeskyQR by panels of 16 columns, head factors four outputs at a time) at
the edges of their classes, through sd.msign and sd.psd_project."""
import numpy as np
import pytest
import torch

import paper_2609_21102_amd as sd
from gpu_util import dev_tensor, host64, rel_fro, workloads
from oracle import muon as omuon
from oracle import psd as opsd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,over", [(1, 16), (16, 1), (7, 17), (13, 12), (3, 29), (31, 2), (32, 32), (49, 14), (63, 1)])
def test_sketch_widths(k, over):
    """r' = 17 to 64; k not a multiple of 4 as well. The singular values are
    those of the float64 oracle to float32 rounding of the panels."""
    case = workloads.small_muon(2, 150, 230, k=min(k, 20), case_id=41)
    out, info = sd.msign(dev_tensor(case.x, "f32"), k, 5, oversample=over, info=True)
    want, oinfo = omuon.msign_deflated(case.x64, k, case.coeffs, oversample=over, power_iters=1, gamma=1.01)
    err = rel_fro(host64(out), want)
    print(f"r'={k + over} k={k}: {err:.2e}", flush=True)
    assert err < 1e-4
    for b in range(2):
        np.testing.assert_allclose(info["s"].cpu().numpy()[b], oinfo.s[b][:k], rtol=1e-5, atol=1e-6 * oinfo.s[b][0])


@pytest.mark.parametrize("k", [17, 24, 25, 31, 32])
def test_ritz_widths(k):
    pc = workloads.small_psd(220, k=k, n_dom=k // 2, case_id=42)
    q = torch.from_numpy(pc.qwarm).cuda()
    out, info = sd.psd_project(torch.from_numpy(pc.z).cuda(), k, pc.steps, q, subspace_iters=2, gamma=pc.gamma,
                               info=True)
    want, basis, oinfo = opsd.psd_project_deflated(pc.z.astype(np.float64), pc.qwarm.astype(np.float64),
                                                   steps=pc.steps, gamma=pc.gamma, subspace_iters=2)
    assert rel_fro(host64(out), want) < 1e-5
    assert rel_fro(host64(q), basis) < 1e-4
    np.testing.assert_allclose(info["ritz"].cpu().numpy(), oinfo.ritz, rtol=1e-4, atol=1e-5 * abs(oinfo.ritz[0]))


@pytest.mark.parametrize("k,over", [(20, 0), (40, 8)])
def test_rank_deficient_panels(k, over):
    """Panels wider than the input's rank: pivots at their floor, finite
    output, flag raised."""
    x = torch.from_numpy(workloads.low_rank(2, 96, 130, 5)).cuda()
    out, info = sd.msign(x, k, 5, oversample=over, info=True)
    assert bool(torch.isfinite(out).all()) and int(info["status"]) & 2
