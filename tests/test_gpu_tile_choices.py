"""GPU parity of the grouped GEMMs at layers chosen for the tiles they take: the 256-row kernel with row, column and K
remainders, experts of no and of few tokens, weight gradients overwritten and added to; 128- and 64-row tiles with K loops
longer than their rings; 32-row tiles with several row blocks of one expert.  tests/test_tile_choices.py (no GPU) checks
that the layers do take these tiles, and that no other tile is without such a layer.  Tolerances as in test_gpu_parity."""
import pytest
import torch

from oracle import modse_oracle as orc
from test_gpu_parity import TOL, check_grads, check_routing, make, max_rel, _runner

pytestmark = pytest.mark.gpu

# name, d, widths, T, dtype, top_k, logit bias, {GEMM: (rows of its tiles, K split)}
BIG, MID = (256, False), (128, False)
CASES = [
    # expert 2 gets no token, expert 5 fewer than one K step of the weight gradients
    ("wgrad_up_256", 416, (1312, 1056, 1248, 1056, 1184, 1120, 1120, 1312), 3392, "bf16", 1, (0, 0, -100, 0, 0, -0.6, 0, 0),
     {"wgrad": BIG, "up": BIG}),
    # more than 128 MB of weight gradients, which go past the caches; expert 2 gets no token
    ("wgrad_256_streamed", 1056, (1312, 1440, 1376, 1344, 1312, 1440, 1344, 1376), 4001, "bf16", 1, (0, 0, -100, 0, 0, 0, 0, 0),
     {"wgrad": BIG}),
    ("up_down_dx_256", 672, (288, 288), 6995, "bf16", 2, None, {"up": BIG, "down": BIG, "dx": BIG}),
    ("dh_dx_256", 416, (224, 160, 288, 288, 160, 288), 14009, "bf16", 2, None, {"dh": BIG, "dx": BIG}),
    ("up_dh_128", 352, (672, 544, 480), 2005, "bf16", 2, None, {"up": MID, "dh": MID}),
    ("down_64", 352, (160, 288), 80, "bf16", 1, None, {"down": (64, False)}),
    # nearly all tokens go to expert 0: four row blocks of 32 where one is expected
    ("down_32_crowded", 160, (2720, 32, 1312, 640), 100, "bf16", 1, (3, 0, 0, 0), {"down": (32, True), "dx": (64, True)}),
    ("wgrad_128_f32", 2528, (352, 352, 352, 480, 352, 352), 775, "f32", 1, None, {"wgrad": MID}),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_parity(case):
    import numpy as np
    from paper_2409_12210_amd.harness import to_host
    name, d, d_ff, T, dtype, k, bias, _ = case
    bias = None if bias is None else np.array(bias, dtype=np.float32)
    inp = make(name, d, d_ff, T, dtype, k, need_dy=True, bias=bias)
    r = _runner(inp, need_bwd=True)
    weights = ("dW_gate", "dW1", "dW3", "dW2")
    for n in weights:
        getattr(r, n).fill_(7.0)
    r.fwd()
    r.bwd()
    got = r.routing_host()
    idx, _ = check_routing(inp, got)
    y_ref = orc.layer_fwd(inp.x, inp.W_gate, inp.W1, inp.W3, inp.W2, d_ff, k, bias, topk_idx=idx)
    assert max_rel(to_host(r.y), y_ref) <= TOL[dtype]
    check_grads(r, inp, idx, TOL[dtype])
    if name.startswith("wgrad") and dtype == "bf16":
        assert got["counts"][2] == 0 and (name != "wgrad_up_256" or 0 < got["counts"][5] < 64)
        assert float(r.dW1[sum(d_ff[:2]):sum(d_ff[:3])].abs().max()) == 0.0
    if name == "down_32_crowded":
        assert got["counts"][0] > 96
    # added to other values: one float32 addition of what was written before
    before = {n: getattr(r, n).clone() for n in weights}
    for n in weights:
        getattr(r, n).normal_()
    old = {n: getattr(r, n).clone() for n in weights}
    r.bwd(accumulate=True)
    torch.cuda.synchronize()
    for n in weights:
        assert torch.equal(getattr(r, n), old[n] + before[n]), n
    # an inference pass (no derivative terms saved)
    q = _runner(inp)
    q.fwd()
    assert max_rel(to_host(q.y), y_ref) <= TOL[dtype]
