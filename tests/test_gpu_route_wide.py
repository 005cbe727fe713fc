"""GPU parity of the routers for more than 16 experts and for the optional gate parts, at the edges of their ranges: one
token, one and four tokens per block, the block-of-32 router with a ragged last block, d that is no multiple of its
column steps, experts masked out by an infinite negative bias.  Integers bit for bit, as in test_gpu_parity."""
import numpy as np
import pytest

from oracle import modse_oracle as orc
from test_gpu_parity import _runner, check_routing, make

pytestmark = pytest.mark.gpu

CASES = [
    ("n17_one_token", 96, 17, 1, "bf16", 2),
    ("n32_512", 544, 32, 512, "bf16", 2),       # last size with one token per block
    ("n64_513_f32", 160, 64, 513, "f32", 2),    # first with four, one token in the last block
    ("n40_4096", 32, 40, 4096, "bf16", 1),
    ("n64_4097", 1056, 64, 4097, "bf16", 2),    # blocks of 32 tokens, d / 32 no multiple of the waves
    ("n33_9001_f32", 288, 33, 9001, "f32", 2),  # more than one group for some blocks
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_route_parity(case):
    name, d, n, T, dtype, k = case
    inp = make(name, d, (32,) * n, T, dtype, k)
    r = _runner(inp)
    r.route()
    check_routing(inp, r.routing_host())


# the permutation with one token per lane (up to 64 tokens and 16 experts), the fused one (up to 4096 tokens) at the edges of
# its blocks of 16, and the scan over block histograms beyond it: several blocks per thread, in registers and (more than 20)
# read twice; one to 64 experts
@pytest.mark.parametrize("n,T,k", [(1, 15, 1), (2, 16, 2), (64, 17, 2), (16, 64, 2), (1, 64, 1), (17, 64, 2), (8, 65, 2),
                                   (3, 4096, 2), (64, 4096, 1), (1, 4097, 1), (2, 9000, 2),
                                   (31, 5003, 2), (64, 12001, 2)])
def test_permutation_parity(n, T, k):
    inp = make("permute", 32, (32,) * n, T, "bf16", k, seed=21)
    r = _runner(inp)
    r.route()
    check_routing(inp, r.routing_host())


@pytest.mark.parametrize("T", [50, 600, 4200], ids=["token", "four_tokens", "block"])
@pytest.mark.parametrize("keep", [(), (0,), (23,), (5, 20)])
def test_masked_experts(T, keep):
    bias = np.full(24, -np.inf, dtype=np.float32)
    bias[list(keep)] = 0.0
    inp = make("masked", 64, (32,) * 24, T, "f32", bias=bias, seed=9 + len(keep))
    r = _runner(inp)
    r.route()
    got = r.routing_host()
    if not keep:  # nothing above -inf: the first two experts, whatever the gate weights
        assert (got["topk_idx"] == [0, 1]).all()
        return
    ref = orc.route(inp.x, inp.W_gate, 24, 2, bias)
    assert (got["topk_idx"] == ref.topk_idx).all()
    assert np.abs(got["topk_w"] - ref.topk_w).max() < 2e-7
