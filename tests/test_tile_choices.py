"""Which tiles the GPU parity cases take (host code, no GPU): a case that is there for a tile takes it, and every tile that
some layer takes is met by a parity case with a K loop longer than any ring, a partial last K step and cut last tiles."""
import random

import pytest

import test_gpu_block_gemm as block
import test_gpu_gate_ext as ext
import test_gpu_parity as parity
import test_gpu_tile_choices as tiles
from choice_probe import GEMMS, choice


@pytest.mark.parametrize("case", tiles.CASES, ids=[c[0] for c in tiles.CASES])
def test_case_takes_the_tiles_it_is_there_for(case):
    name, d, d_ff, T, dtype, k, _, takes = case
    for gemm, (bm, split) in takes.items():
        c = choice(gemm, d, d_ff, k, T, dtype)
        assert (c.bm, c.kchunk > 0) == (bm, split), (gemm, c)
    if name == "wgrad_256_streamed":
        assert 12 * d * sum(d_ff) > 128 << 20


@pytest.mark.parametrize("name", block.LAST_ROWS)
def test_last_rows_case_takes_its_tiles(name):
    _, d, d_ff, T, dtype, k = next(c for c in block.CASES if c[0] == name)
    assert {choice(g, d, d_ff, k, T, dtype).bm for g in ("up", "down", "dh", "dx")} == {block.LAST_ROWS[name][0]}


# d, width of the experts, their number, T, {GEMM: rows of its tiles}: the faster of the tiles where both were measured
F32_FASTER = [
    (32, 32, 8, 256, dict.fromkeys(("up", "down", "dh", "dx"), 32)),
    (64, 64, 8, 256, dict.fromkeys(("up", "down", "dh", "dx"), 32)),
    (256, 256, 8, 512, dict.fromkeys(("up", "down", "dh", "dx"), 32)),
    (256, 256, 8, 1500, dict.fromkeys(("up", "down", "dh", "dx"), 64)),
    (256, 256, 8, 2048, {"up": 32, "dx": 32}),
    (1024, 1024, 8, 100, dict.fromkeys(("up", "down", "dh", "dx"), 32)),
    (1024, 1024, 8, 384, dict.fromkeys(("up", "down", "dh", "dx"), 64)),
    (1024, 1024, 8, 500, dict.fromkeys(("up", "down", "dh", "dx"), 32)),
    (2048, 256, 8, 300, {"up": 32, "dh": 32}),
    (2048, 1280, 4, 200, {"dx": 64}),
]


@pytest.mark.parametrize("case", F32_FASTER, ids=["d%d_f%d_n%d_t%d" % c[:4] for c in F32_FASTER])
def test_f32_layers_of_few_tiles_take_the_faster_ones(case):
    d, f, n, T, takes = case
    assert {g: choice(g, d, [f] * n, 2, T, "f32").bm for g in takes} == takes


def meets_the_edges(gemm, d, d_ff, k, T, dtype, c):
    step = 32 if dtype == "f32" else 64
    if gemm == "wgrad":  # contracts over an expert's rows; its matrices are d_ff x d and d x d_ff
        return T * k / len(d_ff) >= 4 * step and d % c.bn and any(f % c.bm for f in d_ff)
    if gemm in ("up", "dh"):
        depth, columns = [d], d_ff
    else:
        depth, columns = ([min(f, c.kchunk) for f in d_ff] if c.kchunk else d_ff), [d]
    tail = dtype == "f32" or any(f % step for f in ([d] if gemm in ("up", "dh") else d_ff))
    cut = c.bn == 32 or any(n % c.bn for n in columns)  # (widths are multiples of 32: such tiles are never cut)
    return max(depth) >= 4 * step and tail and cut


def test_every_tile_has_a_parity_case():
    cases = [(c[:6], GEMMS) for c in parity.BWD_CASES + ext.LAYER_CASES + block.CASES + tiles.CASES]
    cases += [(c[:6], ("up", "down")) for c in parity.FWD_CASES]
    met = set()
    for (_, d, d_ff, T, dtype, k), gemms in cases:
        for gemm in gemms:
            c = choice(gemm, d, d_ff, k, T, dtype)
            if meets_the_edges(gemm, d, d_ff, k, T, dtype, c):
                met.add((dtype, gemm, c.bm, c.kchunk > 0))
    rng, taken = random.Random(5), {}
    for _ in range(20000):
        n = rng.choice([1, 2, 4, 8, 8, 16, 32, 64])
        d, T, k = 32 * int(2 ** rng.uniform(0, 7)), int(2 ** rng.uniform(0, 15)), min(n, rng.choice([1, 2]))
        d_ff = [32 * int(2 ** rng.uniform(0, 8)) for _ in range(n)]
        dtype = rng.choice(["bf16", "f32"])
        for gemm in GEMMS:
            c = choice(gemm, d, d_ff, k, T, dtype)
            taken[dtype, gemm, c.bm, c.kchunk > 0] = (d, d_ff, T, k)
    assert len(taken) >= 36
    assert set(taken) <= met, {t: taken[t] for t in set(taken) - met}
