"""Tall inputs: the transposing input copy and the last update's transposed
output at tile edges, with pitches and addresses that do and do not allow
16-byte accesses."""
import pytest
import torch

import paper_2609_21102_amd as sd
from gpu_util import dev_tensor, host64, rel_fro, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("m,n", [(3, 1), (129, 128), (130, 63), (136, 64), (192, 72), (300, 129), (513, 200), (640, 256)])
def test_tall_is_the_transpose_of_wide(m, n, dtype, shift):
    """msign(X) = msign(X^T)^T for the undeflated call: the same filter on the
    same canonical layout, so equal bit for bit."""
    x = dev_tensor(workloads.small_muon(2, n, m, dtype=dtype, k=0, case_id=70).x, dtype)
    want = sd.msign(x, 0, 5)
    t = torch.empty(2 * m * n + shift, dtype=x.dtype, device="cuda")[shift:].view(2, m, n)
    t.copy_(x.transpose(1, 2))
    out = torch.zeros(2 * m * n + shift, dtype=x.dtype, device="cuda")[shift:].view(2, m, n)
    sd.msign(t, 0, 5, out=out)
    print(f"{m} x {n} {dtype}: {rel_fro(host64(out), host64(want.transpose(1, 2))):.1e}", flush=True)
    assert torch.equal(out, want.transpose(1, 2))
