"""The backward pass may write dX over x or over dY: every gradient is then, bit for bit, that of separate buffers."""
import pytest
import torch

import test_gpu_gate_ext as gate_ext
from test_gpu_parity import _runner, make

pytestmark = pytest.mark.gpu

# plain gate with dX from whole rows, from the partial sums of a split product, and in float32; with the gate extensions
CASES = [("rows", 256, (128, 384, 192, 320), 700, "bf16", False), ("split", 96, (4128, 96, 3104, 2016), 130, "bf16", False),
         ("f32", 160, (32, 96, 224, 160), 259, "f32", False), ("n24", 64, (32,) * 24, 300, "bf16", False),
         ("ext", 256, (128, 384, 192, 320), 300, "bf16", True)]


@pytest.mark.parametrize("over", ["x", "dY"])
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_dx_over_an_input(case, over):
    name, d, d_ff, T, dtype, ext = case
    if ext:
        _, r, _ = gate_ext.setup(d, d_ff, T, dtype, 2, True, True, True)
    else:
        r = _runner(make(name, d, d_ff, T, dtype, 2, need_dy=True), need_bwd=True)
    names = ["dW_gate", "dW1", "dW3", "dW2"] + (["dW_noise", "dgamma"] if ext else [])
    r.fwd()
    r.bwd()
    want = {n: getattr(r, n).clone() for n in ["dX"] + names}
    r.dX = getattr(r, over)
    r.bwd()
    torch.cuda.synchronize()
    for n in ["dX"] + names:
        assert torch.equal(getattr(r, n), want[n]), n
