"""A workspace sized for a larger batch gives a smaller one the same results, bit for bit, as one of its own size."""
import pytest
import torch

import paper_2409_12210_amd as m
from test_gpu_parity import make, _runner

pytestmark = pytest.mark.gpu

D, D_FF, K = 288, (4128, 96, 3104, 2016), 2


def empty(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("T", [1, 40, 130, 250, 900])
def test_workspace_sized_for_a_larger_batch(T):
    r = _runner(make("workspace", D, D_FF, T, "bf16", K, need_dy=True), need_bwd=True)
    out = []
    for T_ws in (T, 9000):
        r.ws = empty(m.modse_workspace_size(D, D_FF, K, "bf16", T_ws, m.WS_FWD_SAVED))
        r.fwd()
        r.ws = empty(m.modse_workspace_size(D, D_FF, K, "bf16", T_ws, m.WS_BWD))
        r.bwd()
        torch.cuda.synchronize()
        out.append([t.clone() for t in (r.y, r.dX, r.dW_gate, r.dW1, r.dW3, r.dW2)])
    for a, b in zip(*out):
        assert torch.equal(a, b)
