"""fp32 filter products on split fp16 pairs, through the entry points: tile
edges, ranges and the coefficient tables that send them back to the fp32 MFMA."""
import numpy as np
import pytest
import torch

import paper_2609_21102_amd as sd
from gpu_util import dev_tensor, host64, rel_fro, workloads
from oracle import muon as omuon
from oracle import psd as opsd

pytestmark = pytest.mark.gpu

# A product of two split operands is off by at most about 2^-22 of |a||b| per
# term, random in sign, and a float32 sum by 2^-24 per partial sum; through a
# five-step filter the start's rounding grows by 3.4445^5 = 486 in the slowest
# direction: 486 * 2^-24 = 2.9e-5 bounds the relative error of the Muon output.
MUON_TOL = 5e-5
PSD_TOL = 2e-6   # the cubic filter's slope: 1.5^10 = 58, on the bulk alone


@pytest.mark.parametrize("b,m,n", [(1, 32, 33), (1, 128, 129), (2, 64, 700), (9, 300, 260), (5, 640, 768)])
@pytest.mark.parametrize("table", ["muon", "growing", "shrinking"])
def test_muon_tables(b, m, n, table):
    """muon: split products; growing (norms past 4) and shrinking (below 2^-6):
    the fp32 MFMA. 9 x 300 x 260 and 5 x 640 x 768 cross the tile rule."""
    co = {"muon": workloads.muon_coeff_table(5),
          "growing": np.tile(np.float32([6.0, -2.0, 0.25]), (2, 1)),
          "shrinking": np.tile(np.float32([0.05, -0.01, 0.002]), (3, 1))}[table]
    case = workloads.small_muon(b, m, n, k=4, case_id=11)
    out = sd.msign(dev_tensor(case.x, "f32"), 4, len(co), co)
    want, _ = omuon.msign_deflated(case.x64, 4, co, oversample=8, power_iters=1, gamma=1.01)
    err = rel_fro(host64(out), want)
    print(f"{b}x{m}x{n} {table}: {err:.2e}", flush=True)
    assert err < MUON_TOL


@pytest.mark.parametrize("n,k,degree", [(127, 8, 3), (128, 8, 5), (700, 40, 3), (1900, 16, 3), (2432, 16, 3)])
def test_psd_tile_rule(n, k, degree):
    """n = 1900 (120 symmetric tiles) and 2432 (190; the full restore product
    has 361) lie on both sides of the tile rule."""
    pc = workloads.small_psd(n, k=k, case_id=12)
    steps = 2 if n > 1000 else 7
    poly = [[15 / 8, -5 / 4, 3 / 8]] * steps if degree == 5 else None
    q = torch.from_numpy(pc.qwarm).cuda()
    out = sd.psd_project(torch.from_numpy(pc.z).cuda(), k, steps, q, gamma=pc.gamma, poly=poly, poly_degree=degree)
    tab = None if poly is None else np.asarray(poly, np.float32).astype(np.float64)
    want, _, _ = opsd.psd_project_deflated(pc.z.astype(np.float64), pc.qwarm.astype(np.float64), steps=steps,
                                           gamma=pc.gamma, table=tab)
    err = rel_fro(host64(out), want)
    print(f"n={n} k={k} degree={degree}: {err:.2e}", flush=True)
    assert err < PSD_TOL


@pytest.mark.parametrize("e", [-40, -1, 1, 41])
def test_psd_power_of_two_scale_is_exact(e):
    """The filter sees R / theta and the restore product scales R by theta's
    exponent: a power of two on the input is one on the output, bit for bit."""
    pc = workloads.small_psd(300, k=8, case_id=13)
    z = torch.from_numpy(pc.z).cuda()
    outs = [sd.psd_project(zz.contiguous(), 8, 6, torch.from_numpy(pc.qwarm).cuda(), gamma=pc.gamma)
            for zz in (z, z * 2.0 ** e)]
    assert torch.equal(outs[0] * 2.0 ** e, outs[1])
