"""Scratch of the grouped Muon calls: one block for all groups, sliced per
group stream, next to groups that bring their own workspace."""
import pytest
import torch

import paper_2609_21102_amd as sd
from gpu_util import dev_tensor, workloads

pytestmark = pytest.mark.gpu

SHAPES = [(3, 64, 200), (1, 300, 128), (2, 129, 130), (4, 40, 90), (1, 700, 260), (2, 64, 200), (5, 33, 32)]


@pytest.mark.parametrize("own", [(), (1,), tuple(range(len(SHAPES)))], ids=["none", "one", "all"])
def test_groups_share_slices(own):
    """Seven groups on three streams (so slices are reused, by smaller and by
    larger groups) equal their single calls bit for bit, twice in a row."""
    xs = [dev_tensor(workloads.small_muon(*s, dtype="bf16", k=4, case_id=21 + i).x, "bf16")
          for i, s in enumerate(SHAPES)]
    want = [sd.msign(x, 4, 5) for x in xs]
    groups, keep = [], []
    for i, x in enumerate(xs):
        g = {"x": x, "k": 4, "steps": 5}
        groups.append(g)
    arr = (sd.MsignGroup * len(xs))()
    outs = [torch.empty_like(x) for x in xs]
    for i, x in enumerate(xs):
        o = sd.msign_opts()
        if i in own:
            ws = torch.empty(sd.msign_workspace_bytes(*x.shape, 4), dtype=torch.uint8, device="cuda")
            o.workspace, o.workspace_bytes = ws.data_ptr(), ws.numel()
            keep.append(ws)
        keep.append(o)
        arr[i] = sd.MsignGroup(*x.shape, 4, 5, None, sd.SD_DTYPE_BF16, x.data_ptr(), outs[i].data_ptr(),
                               sd.ctypes.pointer(o))
    for _ in range(2):
        for y in outs:
            y.zero_()
        assert sd.lib().sd_msign_groups(len(xs), arr, sd._stream(None)) == sd.SD_OK
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(outs, want))
    assert all(torch.equal(a, b) for a, b in zip(sd.msign_groups(groups), want))


def test_small_workspace_of_a_group_is_refused():
    """A group's own workspace that is too small: SD_ERR_WORKSPACE."""
    x = dev_tensor(workloads.small_muon(2, 64, 200, dtype="bf16", k=4).x, "bf16")
    arr, keep = (sd.MsignGroup * 2)(), []
    for i in range(2):
        o = sd.msign_opts()
        ws = torch.empty(1024 if i else sd.msign_workspace_bytes(2, 64, 200, 4), dtype=torch.uint8, device="cuda")
        o.workspace, o.workspace_bytes = ws.data_ptr(), ws.numel()
        y = torch.empty_like(x)
        keep += [o, ws, y]
        arr[i] = sd.MsignGroup(2, 64, 200, 4, 5, None, sd.SD_DTYPE_BF16, x.data_ptr(), y.data_ptr(),
                               sd.ctypes.pointer(o))
    assert sd.lib().sd_msign_groups(2, arr, sd._stream(None)) == -5
    torch.cuda.synchronize()
