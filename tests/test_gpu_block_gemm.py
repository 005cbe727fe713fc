"""GPU parity of the grouped GEMMs with small tiles (one workgroup per tile): forward and every gradient against the
fp64 CPU oracle, at sizes whose row, column and K remainders fall on every side of the tile edges.  Tolerances are those
of the layer's parity tests: max|out - ref| <= tol * max|ref|, 1e-4 (fp32) and 2e-2 (bf16 storage of the activations)."""
import pytest

import test_gpu_gate_ext as gate_ext
from oracle import modse_oracle as orc
from test_gpu_parity import TOL, check_grads, check_routing, make, max_rel, _runner

pytestmark = pytest.mark.gpu

# d and the widths are odd multiples of 32
WIDE = tuple(32 * w for w in (21, 27, 17, 31, 24, 24, 23, 29))

CASES = [
    # 64 x 64 tiles, several rounds of them
    ("f32_many_tiles_64", 544, WIDE, 6205, "f32", 2),
    # rounds of 128-row tiles that fit: the forward and data-gradient products; the weight gradients
    ("f32_tall", 736, (864, 992, 736, 992), 30001, "f32", 1),
    ("f32_wide", 992, (992, 1120) * 8, 200, "f32", 2),
    ("f32_tiles_64_last_rows", 544, WIDE, 1324, "f32", 2),
    ("f32_narrow", 160, (32, 96, 224, 160), 259, "f32", 2),
    ("f32_one_row", 64, (32, 96), 1, "f32", 1),
    # 32 x 32 tiles whose waves share out K: loops as long as the ring and longer
    ("f32_tiles_32_four_steps", 128, (32, 128, 64), 95, "f32", 2),
    ("f32_tiles_32_four_steps_last_rows", 128, (32, 128, 64), 191, "f32", 2),
    ("f32_tiles_32_long_loops", 416, (672, 32, 352, 544), 130, "f32", 2),
    ("f32_tiles_32_long_loops_last_rows", 416, (672, 32, 352, 544), 120, "f32", 2),
    ("f32_split", 160, (4128, 2048, 1952, 672), 97, "f32", 2),
    # bf16, the products with d columns: K split into chunks (widths of 1 to 7 chunks, the last ones ragged) over 32-row
    # tiles (one row), 64-row tiles (32 and 48 mean rows per expert) and 128-row ones (125); 128- and 32-row tiles, unsplit
    ("bf16_one_row", 96, (32, 2720), 1, "bf16", 2),
    ("bf16_rows_32", 96, (2720, 32, 1312, 640), 64, "bf16", 2),
    ("bf16_rows_64", 160, (4128, 2048, 1952, 672), 97, "bf16", 2),
    ("bf16_rows_128", 224, (4128, 96, 3104, 2016), 250, "bf16", 2),
    ("bf16_rows_129", 288, (96, 160, 224, 288) * 4, 1033, "bf16", 2),
    ("bf16_few_rows_many_experts", 64, (32,) * 64, 200, "bf16", 1),
    # one row block per expert, whose K loops start anywhere: 33 and 34 K steps, the last ones partial; dX with both operand
    # pairs in one loop (many experts: not split)
    ("bf16_one_block_33_steps", 2080, (2144, 96, 2080, 1184), 60, "bf16", 2),
    ("bf16_one_block_17_steps", 1056, (1056, 1120, 992, 1184) * 8, 300, "bf16", 2),
]
# cases that are there for the last row block of an expert: rows of the tiles of all four products; rows that it has, each at
# one expert at least
LAST_ROWS = {
    "f32_tiles_64_last_rows": (64, {1, 55}),
    "f32_tiles_32_four_steps_last_rows": (32, {1, 30, 31}),
    "f32_tiles_32_long_loops_last_rows": (32, {1, 18, 30, 31}),
}


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_fwd_and_grads(case):
    from paper_2409_12210_amd.harness import to_host
    name, d, d_ff, T, dtype, k = case
    inp = make(name, d, d_ff, T, dtype, k, need_dy=True)
    r = _runner(inp, need_bwd=True)
    r.fwd()
    r.bwd()
    got = r.routing_host()
    idx, _ = check_routing(inp, got)
    if name in LAST_ROWS:
        bm, rows = LAST_ROWS[name]
        assert rows <= {int(c) % bm for c in got["counts"]}
    y_ref = orc.layer_fwd(inp.x, inp.W_gate, inp.W1, inp.W3, inp.W2, d_ff, k, topk_idx=idx)
    assert max_rel(to_host(r.y), y_ref) <= TOL[dtype]
    g = check_grads(r, inp, idx, TOL[dtype])
    r.bwd(accumulate=True)
    for n in ("dW1", "dW3", "dW2", "dW_gate"):
        assert max_rel(to_host(getattr(r, n)), 2 * getattr(g, n)) <= TOL[dtype], n


@pytest.mark.parametrize("T", [40, 250])
def test_workspace_without_room_for_partial_sums(T):
    """The smallest workspace that is accepted lacks the partial sums of the split products.  It serves all the same,
    unsplit, with results inside the same tolerance."""
    import torch
    import paper_2409_12210_amd as m
    from paper_2409_12210_amd.harness import to_host
    d, d_ff, k = 288, (4128, 96, 3104, 2016), 2
    inp = make("short_ws", d, d_ff, T, "bf16", k, need_dy=True)
    r = _runner(inp, need_bwd=True)
    slab = T * k * d * 4
    for which, call in ((m.WS_FWD_SAVED, r.fwd), (m.WS_BWD, r.bwd)):
        full = m.modse_workspace_size(d, d_ff, k, "bf16", T, which)
        refused, accepted = 0, full
        while accepted - refused > 256:
            r.ws = torch.empty((refused + accepted) // 2, dtype=torch.uint8, device="cuda")
            try:
                call()
                accepted = r.ws.numel()
            except m.ModseError as e:
                assert e.code == 3
                refused = r.ws.numel()
        assert full - accepted > slab
        r.ws = torch.empty(accepted, dtype=torch.uint8, device="cuda")
        call()
    idx, _ = check_routing(inp, r.routing_host())
    y_ref = orc.layer_fwd(inp.x, inp.W_gate, inp.W1, inp.W3, inp.W2, d_ff, k, topk_idx=idx)
    assert max_rel(to_host(r.y), y_ref) <= TOL["bf16"]
    check_grads(r, inp, idx, TOL["bf16"])


@pytest.mark.parametrize("case", [
    ("ext_split", 96, (4128, 96, 3104, 2016), 130, "bf16", 2),   # dX in partial sums, both gate extensions
    ("ext_many_tokens", 32, (32, 64, 32, 96), 65633, "bf16", 2),  # several groups of tokens per block of the router's backward
], ids=lambda c: c[0])
def test_gate_ext(case):
    gate_ext.test_layer_fwd_bwd_ext_parity(case, True, True)


def test_many_tokens_plain_gate():
    """Chunks of several token groups in the router's weight gradient, columns that do not fill a slab."""
    T, d, d_ff, k = 65633, 32, (32, 64, 96), 2
    inp = make("many_tokens", d, d_ff, T, "f32", k, need_dy=True)
    r = _runner(inp, need_bwd=True)
    r.fwd()
    r.bwd()
    idx, _ = check_routing(inp, r.routing_host())
    check_grads(r, inp, idx, TOL["f32"])
