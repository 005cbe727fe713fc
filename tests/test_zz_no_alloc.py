"""modse_route_static, the entry point that allocates nothing (its scratch is a device array inside the
library), against modse_route on the same inputs: every routing output bit for bit, on two calls in a row
that share the array, the second with fewer tokens.  Collected last on purpose."""
import numpy as np
import pytest
import torch

import paper_2409_12210_amd as m
import workloads as wl
from paper_2409_12210_amd.harness import LayerRunner, to_host

pytestmark = pytest.mark.gpu

FIELDS = ("topk_idx", "topk_w", "counts", "offsets", "row_of", "src_of", "near_tie_count")

# (name, d_model, d_ff, dtype, top_k, T of the first call, T of the second call)
CASES = [
    ("blocks_then_tokens", 256, (128, 384, 192, 320, 224, 288, 256, 256), "f32", 2, 5000, 50),
    ("bf16_ragged", 512, (96, 416, 160, 352, 224, 288, 256, 256), "bf16", 2, 20001, 1237),
    ("n64", 64, (32,) * 64, "f32", 2, 3000, 200),
    ("top1_tokens", 256, (128, 384, 192, 320), "bf16", 1, 64, 1),
]


def route_both(name, d, d_ff, dtype, k, T, seed):
    cfg = wl.LayerConfig(name, d, tuple(d_ff), k, T, dtype, seed=seed, dy_seed=seed + 1)
    r = LayerRunner.from_inputs(wl.make_inputs(cfg))
    r.route()
    want = r.routing_host()
    other = m.Routing.empty(T, len(d_ff), k, "cuda")
    for f in FIELDS:  # stale contents must not survive
        getattr(other, f).fill_(-7)
    before = torch.cuda.memory_allocated()
    m.modse_route_static(d, list(d_ff), k, dtype, T, r.x, r.W_gate, r.bias, other)
    torch.cuda.synchronize()
    assert torch.cuda.memory_allocated() == before
    for f in FIELDS:
        got = to_host(getattr(other, f))
        assert got.dtype == want[f].dtype and got.shape == want[f].shape, f
        assert np.array_equal(got.view(np.int32), want[f].view(np.int32)), (name, T, f)


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_route_static_matches_route_on_two_calls_in_a_row(case):
    name, d, d_ff, dtype, k, T_first, T_second = case
    route_both(name, d, d_ff, dtype, k, T_first, seed=11)
    route_both(name, d, d_ff, dtype, k, T_second, seed=12)


# bf16, more than 16 experts, from 1536 or 2049 tokens on: routers that want room for W_gate's columns, whose 1 MiB would not fit
# behind the scratch of the last two.  Values that cancel, so that the order of the sums shows in the gate weights.
@pytest.mark.parametrize("d,n,T", [(256, 64, 1700), (512, 24, 4500), (8192, 64, 2000), (4096, 64, 50001)])
def test_route_static_takes_the_same_router(d, n, T):
    gen = torch.Generator(device="cuda").manual_seed(d + T)
    x = torch.randn((T, d), device="cuda", generator=gen).bfloat16()
    W = (0.02 * torch.randn((d, n), device="cuda", generator=gen)).bfloat16()
    x[:, 0] = x[:, d - 1] = 2.0 ** 28
    W[d - 1] = -W[0]
    routings = [m.Routing.empty(T, n, 2, "cuda") for _ in range(2)]
    ws = torch.empty(m.modse_workspace_size(d, [32] * n, 2, "bf16", T, m.WS_FWD), dtype=torch.uint8, device="cuda")
    m.modse_route(d, [32] * n, 2, "bf16", T, x, W, None, routings[0], ws)
    m.modse_route_static(d, [32] * n, 2, "bf16", T, x, W, None, routings[1])
    for f in FIELDS:
        want, got = getattr(routings[0], f), getattr(routings[1], f)
        assert torch.equal(got.view(torch.int32), want.view(torch.int32)), f


def test_route_static_rejects_more_tokens_than_the_array_serves():
    d_ff = [32] * 64
    T = 1 << 18
    x = torch.zeros(8, device="cuda")
    r = m.Routing.empty(8, 64, 2, "cuda")
    code = m.modse_route_static(64, d_ff, 2, "f32", T, x, x, None, r, raise_on_error=False)
    assert code == 3 and "workspace" in m.modse_status_string(code)
    with pytest.raises(m.ModseError):
        m.modse_route_static(64, d_ff, 2, "f32", T, x, x, None, r)
