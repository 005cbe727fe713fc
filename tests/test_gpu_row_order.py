"""What a token's output and gradient depend on: its own row and the size of the batch.  Neither its place among an expert's
rows nor the other tokens (how many rows an expert has, which tiles they fill, which workgroups take these) changes a bit of
either, in any tile shape of the grouped GEMMs."""
import pytest
import torch

from choice_probe import choice
from test_gpu_parity import make, _runner

pytestmark = pytest.mark.gpu

# name, d, widths, T, dtype, top_k, {GEMM: rows of its tiles}
CASES = [
    ("several_blocks_of_128", 672, (672, 544, 480), 2005, "bf16", 2, {"up": 128, "dh": 128}),
    ("products_with_d_columns_of_128", 1056, (1056, 1120, 992, 1184) * 4, 1205, "bf16", 2, {"down": 128, "dx": 128}),
    ("one_block_of_64", 2080, (2144, 96, 2080, 1184), 60, "bf16", 2, {"up": 64, "dx": 64}),
    ("blocks_of_32", 2080, (2720, 1312, 640, 2080), 50, "bf16", 2, {"down": 32}),
    ("split_blocks_of_128", 224, (4128, 96, 3104, 2016), 250, "bf16", 2, {"down": 128, "dx": 128}),
    ("blocks_of_256", 672, (288,) * 4, 14001, "bf16", 2, {"down": 256, "dh": 256, "dx": 256}),
    ("up_256_top1", 416, (1312, 1056, 1248, 1056, 1184, 1120, 1120, 1312), 3392, "bf16", 1, {"up": 256}),
    ("f32_blocks_of_32", 416, (672, 32, 352, 544), 130, "f32", 2, {"up": 32, "dx": 32}),
    ("f32_larger_blocks", 544, (672, 864, 544, 992) * 2, 3001, "f32", 2, {"up": 64}),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_rows_do_not_depend_on_their_neighbours(case):
    name, d, d_ff, T, dtype, k, takes = case
    for gemm, bm in takes.items():
        assert choice(gemm, d, d_ff, k, T, dtype).bm == bm, gemm
    inp = make(name, d, d_ff, T, dtype, k, need_dy=True)
    r = _runner(inp, need_bwd=True)
    half = T // 2

    def outputs():
        r.fwd()
        r.bwd()
        torch.cuda.synchronize()
        return r.y.clone(), r.dX.clone(), r.routing.counts.cpu()

    y, dX, counts = outputs()
    # the second half of the batch becomes copies of token 0: two experts get most of the rows, the others fewer
    for t in (r.x, r.dY):
        t[half:] = t[0]
    y2, dX2, counts2 = outputs()
    assert int(counts2.max()) > half >= 1 and not torch.equal(counts, counts2)
    for a, b, what in ((y, y2, "y"), (dX, dX2, "dX")):
        assert torch.equal(b[half:], a[:1].expand(T - half, d)), what + " of equal tokens"
        assert torch.equal(b[:half], a[:half]), what + " of tokens among others"
