"""Backward passes of layers of small tiles, whose dX, weight gradients and router's weight gradient share a launch: every
combination of their tiles, with the router's part (plain gate) and without it (gate with a noise term), d that ends inside a tile
and batches that end inside a block of tokens.  Tolerances as in test_gpu_parity; a gradient added to other values is one float32
addition of what is written otherwise, bit for bit."""
import pytest
import torch

from choice_probe import choice
from test_gpu_parity import TOL, _runner, check_grads, check_routing, make

# name, d, widths, T, dtype, top_k, (rows of dX's tiles, K split), rows of the weight gradients' tiles
CASES = [
    ("f32_32_64", 544, (512, 96, 160), 109, "f32", 2, (32, False), 64),
    ("f32_64_64", 480, (1088, 1120), 765, "f32", 2, (64, False), 64),
    ("f32_64_split_64", 32, (544, 2592), 299, "f32", 1, (64, True), 64),
    ("f32_64_split_128", 608, (3040, 1344, 2080, 2336, 3328), 12, "f32", 1, (64, True), 128),
    ("bf16_64_128", 544, (1088, 64), 48, "bf16", 2, (64, False), 128),
    ("bf16_64_split_128", 96, (1728, 2144, 2144), 52, "bf16", 2, (64, True), 128),
    ("bf16_128_128", 288, (352, 416, 32), 897, "bf16", 1, (128, False), 128),
    ("bf16_128_split_128", 32, (2304, 2208), 813, "bf16", 1, (128, True), 128),
    ("bf16_128_split_256", 416, (2336, 3648, 3552), 684, "bf16", 2, (128, True), 256),
]
IDS = [c[0] for c in CASES]


@pytest.mark.parametrize("case", CASES, ids=IDS)
def test_case_takes_its_tiles(case):
    _, d, d_ff, T, dtype, k, dx, wgrad = case
    c = choice("dx", d, d_ff, k, T, dtype)
    assert (c.bm, c.kchunk > 0) == dx and choice("wgrad", d, d_ff, k, T, dtype).bm == wgrad


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=IDS)
def test_parity(case):
    _, d, d_ff, T, dtype, k, _, _ = case
    inp = make("one_launch", d, d_ff, T, dtype, k, need_dy=True)
    r = _runner(inp, need_bwd=True)
    weights = ("dW_gate", "dW1", "dW3", "dW2")
    for n in weights:
        getattr(r, n).fill_(7.0)
    r.fwd()
    r.bwd()
    idx, _ = check_routing(inp, r.routing_host())
    check_grads(r, inp, idx, TOL[dtype])
    before = {n: getattr(r, n).clone() for n in weights}
    old = {n: getattr(r, n).normal_().clone() for n in weights}
    r.bwd(accumulate=True)
    torch.cuda.synchronize()
    for n in weights:
        assert torch.equal(getattr(r, n), old[n] + before[n]), n


@pytest.mark.gpu
@pytest.mark.parametrize("case", [CASES[0], CASES[5], CASES[6]], ids=[IDS[0], IDS[5], IDS[6]])
def test_gate_with_noise_term(case):
    import test_gpu_gate_ext as ext
    _, d, d_ff, T, dtype, k, _, _ = case
    ext.test_layer_fwd_bwd_ext_parity(("one_launch", d, d_ff, T, dtype, k), True, True)
