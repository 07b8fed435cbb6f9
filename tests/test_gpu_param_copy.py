"""Gather and scatter of parameter lists: tall and wide members, pitches and
addresses that do and do not allow 16-byte accesses, partial tiles."""
import pytest
import torch

import paper_2609_21102_amd as sd
from gpu_util import workloads

pytestmark = pytest.mark.gpu

SHAPES = [(1, 3), (5, 5), (63, 65), (64, 128), (65, 136), (72, 129), (128, 192), (130, 70)]


def put(x, dtype, shift):
    """`x` on the GPU, `shift` elements past a 16-byte boundary."""
    t = torch.empty(x.size + shift, dtype=dtype, device="cuda")[shift:].view(x.shape)
    return t.copy_(torch.from_numpy(x))


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_members_match_single_calls(dtype, shift):
    """Each shape as two wide and two tall members: every output equals the
    member's own call up to the output's rounding (one unit of bfloat16 where a
    product's tiling differs; a misplaced element is an error of order one)."""
    xs = []
    for i, (m, n) in enumerate(SHAPES):
        w = workloads.small_muon(4, m, n, k=0, case_id=60 + i).x
        xs += [put(w[0].copy(), dtype, shift), put(w[1].T.copy(), dtype, shift), put(w[2].copy(), dtype, 0),
               put(w[3].T.copy(), dtype, 0)]
    outs = [put(torch.zeros(x.shape).numpy(), dtype, shift) for x in xs]
    sd.msign_params(xs, 0, 5, outs=outs)
    again = [x.clone() for x in xs]
    sd.msign_params(again, 0, 5, outs=again)   # in place
    tol = 2.0 ** -8 if dtype == torch.bfloat16 else 1e-5
    for x, y, z in zip(xs, outs, again):
        want = sd.msign(x[None].contiguous(), 0, 5)[0].double()
        err = float(torch.linalg.norm(y.double() - want) / torch.linalg.norm(want))
        print(f"{tuple(x.shape)} {dtype}: {err:.1e}", flush=True)
        assert err <= tol and torch.equal(y, z)
