"""GPU parity of the grouped GEMMs with small tiles (one workgroup per tile): forward and every gradient against the
fp64 CPU oracle, at sizes whose row, column and K remainders fall on every side of the tile edges.  Tolerances are those
of the layer's parity tests: max|out - ref| <= tol * max|ref|, 1e-4 (fp32) and 2e-2 (bf16 storage of the activations)."""
import pytest

from oracle import modse_oracle as orc
from test_gpu_parity import TOL, check_grads, check_routing, make, max_rel, _runner

pytestmark = pytest.mark.gpu

# enough tiles for 128 x 128 ones in every GEMM; d and the widths are odd multiples of 32
WIDE = tuple(32 * w for w in (21, 27, 17, 31, 24, 24, 23, 29))

CASES = [
    ("f32_tiles_128", 544, WIDE, 6205, "f32", 2),
    ("f32_tiles_64", 160, (32, 96, 224, 160), 259, "f32", 2),       # 64 x 64 tiles, one row past two of them
    ("f32_one_row", 64, (32, 96), 1, "f32", 1),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_fwd_and_grads(case):
    from paper_2409_12210_amd.harness import to_host
    name, d, d_ff, T, dtype, k = case
    inp = make(name, d, d_ff, T, dtype, k, need_dy=True)
    r = _runner(inp, need_bwd=True)
    r.fwd()
    r.bwd()
    idx, _ = check_routing(inp, r.routing_host())
    y_ref = orc.layer_fwd(inp.x, inp.W_gate, inp.W1, inp.W3, inp.W2, d_ff, k, topk_idx=idx)
    assert max_rel(to_host(r.y), y_ref) <= TOL[dtype]
    g = check_grads(r, inp, idx, TOL[dtype])
    r.bwd(accumulate=True)
    assert max_rel(to_host(r.dW1), 2 * g.dW1) <= TOL[dtype]
    assert max_rel(to_host(r.dW2), 2 * g.dW2) <= TOL[dtype]
