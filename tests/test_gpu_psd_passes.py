"""The passes around the filter of the PSD projection at the edges of their
variants: Lanczos steps by length and number of steps, the one-work-group
eigenproblem of wide bases up to 64, the output pass by tile pairs, and the
ADMM's padded shift."""
import numpy as np
import pytest
import torch

import paper_2609_21102_amd as sd
import workloads
from oracle import psd as opsd
from tests.gpu_util import host64, rel_fro, say

pytestmark = pytest.mark.gpu


def offset(a: np.ndarray) -> torch.Tensor:
    """`a` on the GPU, 4 bytes past a 16-byte boundary."""
    t = torch.empty(a.size + 1, dtype=torch.float32, device="cuda")[1:].view(a.shape)
    return t.copy_(torch.from_numpy(a))


@pytest.mark.parametrize("n,steps", [(1, 20), (130, 4), (2048, 20), (2048, 25), (2049, 12), (2049, 13), (4096, 20),
                                     (4097, 5), (8064, 20), (1000, 64), (3000, 64), (4200, 64)])
def test_lanczos_steps(n, steps):
    """Both ends of each length's variant, with fewer and more steps than the
    basis vectors it keeps; theta (no deflation, no filter steps) against the
    float64 recurrence of the oracle. The estimate is a converged Ritz value or
    has a full-length recurrence behind it, so float32 storage of the basis
    enters it squared: 1e-5 as for the longer steps."""
    z = workloads.sym_gaussian(n, case_id=1)
    say(f"lanczos n={n} steps={steps}")
    out, info = sd.psd_project(torch.from_numpy(z).cuda(), 0, 0, None, lanczos_steps=steps, info=True)
    z64 = z.astype(np.float64)
    want = opsd.lanczos_scale(lambda x: z64 @ (z64 @ x), n, 0, steps)
    assert abs(float(info["theta"]) - want) <= 1e-5 * want


@pytest.mark.parametrize("k", [33, 48, 63, 64, 65])
def test_wide_ritz_widths(k):
    """One work-group up to K = 64, block Jacobi from 65."""
    case = workloads.small_psd(260, k=k, n_dom=k // 2, case_id=44)
    z, q = torch.from_numpy(case.z).cuda(), torch.from_numpy(case.qwarm).cuda()
    out, info = sd.psd_project(z, k, case.steps, q, subspace_iters=2, gamma=case.gamma, info=True)
    want, basis, oinfo = opsd.psd_project_deflated(case.z.astype(np.float64), case.qwarm.astype(np.float64),
                                                   steps=case.steps, gamma=case.gamma, subspace_iters=2)
    assert int(info["status"]) == 0
    assert rel_fro(host64(out), want) < 1e-4 and rel_fro(host64(q), basis) < 1e-4
    np.testing.assert_allclose(info["ritz"].cpu().numpy(), oinfo.ritz, rtol=1e-4, atol=1e-5 * abs(oinfo.ritz[0]))


@pytest.mark.parametrize("k", [40, 70])
def test_wide_ritz_flags_nan(k):
    """An eigenproblem that cannot converge sets the flag on both routes."""
    case = workloads.small_psd(200, k=k, case_id=45)
    z = case.z.copy()
    z[3, 5] = z[5, 3] = np.nan
    _, info = sd.psd_project(torch.from_numpy(z).cuda(), k, 5, torch.from_numpy(case.qwarm).cuda(), info=True)
    assert int(info["status"]) & 8


@pytest.mark.parametrize("n,k", [(1, 0), (2, 1), (63, 4), (64, 4), (65, 16), (130, 8), (131, 17), (132, 40), (1100, 32)])
@pytest.mark.parametrize("aligned", [True, False])
def test_output_tiles(n, k, aligned):
    """Rows that are and are not whole 16-byte pieces, from aligned and
    unaligned buffers, one tile and several bands of tiles."""
    case = workloads.small_psd(n, k=max(k, 1), n_dom=min(4, max(k, 1), n), case_id=46)
    z = torch.from_numpy(case.z).cuda() if aligned else offset(case.z)
    out = torch.empty_like(z) if aligned else offset(np.zeros_like(case.z))
    q = torch.from_numpy(case.qwarm).cuda() if k else None
    sd.psd_project(z, k, case.steps, q, subspace_iters=2, gamma=case.gamma, out=out)
    z64 = case.z.astype(np.float64)
    if k:
        want = opsd.psd_project_deflated(z64, case.qwarm.astype(np.float64), steps=case.steps, gamma=case.gamma,
                                         subspace_iters=2)[0]
    else:
        want = opsd.psd_project(z64, steps=case.steps)[0]
    assert rel_fro(host64(out), want) < 1e-4
    assert torch.equal(out, out.T)


@pytest.mark.parametrize("n,aligned", [(128, True), (130, True), (133, True), (132, False), (256, True)])
def test_admm_padding(n, aligned):
    """Lengths that are multiples of 128, of 4 and of neither; the padding of
    the shifted matrix stays zero over the iterations. Each iteration adds at
    most one projection's tolerance to the state."""
    from oracle import admm as oadmm
    case = workloads.planted_maxcut(n, case_id=4)
    put = (lambda a: torch.from_numpy(a).cuda()) if aligned else offset
    q = torch.from_numpy(np.ascontiguousarray(case.basis0, dtype=np.float32)).cuda()
    zero = np.zeros((n, n), np.float32)
    X, S, y, eta, _ = sd.admm_diag(put(case.c), torch.from_numpy(case.b).cuda(), 4, case.k, q, X=put(zero),
                                   S=put(zero), warmup=4, tau=0.1, window=case.window)
    proj = oadmm.DeflatedProjector(case.basis0.astype(np.float64), tau=0.1, window=case.window, warmup=4, mode="exact")
    xo, so, yo, etas = oadmm.admm_diag(case.c.astype(np.float64), case.b.astype(np.float64), 4, proj,
                                       x=zero.astype(np.float64), s=zero.astype(np.float64), y=np.zeros(n))
    assert max(rel_fro(host64(X), xo), rel_fro(host64(S), so), rel_fro(host64(y), yo)) < 4e-4
