"""The bf16 path's grouped fp16 filter through sd.msign: group sizes, the
l_pad = 2 s_pad edge, tables without a quintic term and tables outside its
range, against the float64 filter and the bf16 contract's own error."""
import numpy as np
import pytest

import paper_2609_21102_amd as sd
from gpu_util import dev_tensor, host64, rel_fro, workloads
from oracle import muon as omuon

pytestmark = pytest.mark.gpu

CLASSIC = np.tile(np.float32([1.5, -0.5, 0.0]), (6, 1))
GROWING = np.tile(np.float32([6.0, -2.0, 0.25]), (2, 1))   # leaves the fp16 form's range


def check(case, k, table, **kw):
    out = host64(sd.msign(dev_tensor(case.x, "bf16"), k, len(table), table, **kw))
    args = dict(oversample=8, power_iters=1, gamma=kw.get("gamma", 1.01), restore=kw.get("restore", "padded"))
    exact, _ = omuon.msign_deflated(case.x64, k, table, mode="exact", **args)
    contract, _ = omuon.msign_deflated(case.x64, k, table, mode="bf16", **args)
    for b in range(len(out)):
        err, own = rel_fro(out[b], exact[b]), rel_fro(contract[b], exact[b])
        print(f"{case.name} k={k} {len(table)} steps: {err:.2e}, bf16 contract {own:.2e}", flush=True)
        # no worse than bf16 products; bf16 output rounding alone is 1.7e-3
        assert err < max(own, 2.5e-3)


@pytest.mark.parametrize("b,m,n", [(2, 64, 256), (1, 128, 255), (1, 130, 512), (1, 130, 513), (2, 700, 33), (3, 256, 520)])
@pytest.mark.parametrize("steps", [1, 2, 3, 4, 5, 8])
def test_group_sizes(b, m, n, steps):
    case = workloads.small_muon(b, m, n, dtype="bf16", k=4, case_id=31)
    check(case, 4, workloads.muon_coeff_table(steps))


@pytest.mark.parametrize("table", [CLASSIC, workloads.polar_express_like_table(0, 8), GROWING],
                         ids=["cubic", "pe8", "growing"])
@pytest.mark.parametrize("k,restore", [(0, "padded"), (4, "padded"), (4, "explicit")])
def test_tables(table, k, restore):
    case = workloads.small_muon(2, 96, 400, dtype="bf16", k=4, case_id=32)
    check(case, k, table, restore=restore)


@pytest.mark.parametrize("b", [2, 11, 26])
def test_tile_rules(b):
    """384 x 768 (6 tiles of 128 x 128 a matrix): 12, 66 and 156 tiles take the
    three tile forms; every matrix equals itself in a batch of one."""
    case = workloads.small_muon(1, 384, 768, dtype="bf16", k=4, case_id=33)
    x = dev_tensor(case.x, "bf16")
    one = sd.msign(x, 4, 5)
    sk = sd.sketch(1, 384, 12)
    many = sd.msign(x.expand(b, -1, -1).contiguous(), 4, 5, sketch=sk.expand(b, -1, -1).contiguous())
    for i in range(b):
        assert rel_fro(host64(many[i]), host64(one[0])) < 2e-6 or bool((many[i] == one[0]).all())
