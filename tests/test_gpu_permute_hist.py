"""The permutation of batches of more than 4096 tokens: over the block histograms in one launch, or by scan and scatter, at the edges
between the two, with one counter column per thread and with many, without rows (routing calls) and with them (layer calls, whose
outputs must be a small batch's, row by row).  Integers bit for bit."""
import pytest
import torch

from choice_probe import permute_by_hist
from test_gpu_parity import _runner, check_routing, make

# experts, tokens, top_k, one launch
ROUTE = [(64, 16128, 2, True), (64, 16129, 2, False), (1, 8193, 1, False), (8, 116481, 2, False), (7, 131073, 1, False), (37, 4127, 2, True),
         (1, 8192, 1, True), (8, 8161, 2, True), (48, 8193, 2, False), (49, 8193, 1, True)]
# experts, d, tokens, top_k, dtype, one launch
LAYER = [(64, 32, 16128, 2, "bf16", True), (64, 32, 16129, 2, "bf16", False), (17, 64, 12288, 1, "bf16", True), (36, 64, 12289, 2, "f32", False),
         (37, 32, 16384, 2, "f32", True), (37, 32, 16385, 2, "f32", False), (16, 64, 8193, 2, "bf16", False), (3, 1024, 9001, 2, "f32", True),
         (3, 992, 9001, 2, "f32", False), (2, 2048, 32768, 2, "bf16", True), (2, 2048, 32769, 2, "bf16", False),
         (2, 2048, 8193, 1, "bf16", False)]


def test_cases_take_the_launch_they_are_there_for():
    for n, T, k, one in ROUTE:
        assert permute_by_hist(32, n, k, T, "bf16", False) == one, (n, T, k)
    for n, d, T, k, dtype, one in LAYER:
        assert permute_by_hist(d, n, k, T, dtype, True) == one, (n, d, T, k, dtype)


# both measured: d, experts, top_k, tokens, whether rows are copied, the faster one
@pytest.mark.parametrize("d,n,k,T,rows,one", [
    (256, 1, 1, 400000, False, False), (256, 2, 2, 262144, False, False), (256, 8, 2, 16384, False, False), (256, 8, 2, 116000, False, False),
    (256, 16, 2, 32768, False, False), (256, 32, 2, 31000, False, False), (256, 64, 2, 12288, False, True), (256, 8, 2, 8192, False, True),
    (2048, 1, 1, 32768, True, False), (2048, 8, 2, 32768, True, True), (2048, 8, 2, 65536, True, False), (256, 8, 2, 32768, True, False),
    (2048, 20, 1, 20000, True, False), (2048, 64, 2, 12000, True, True), (256, 24, 2, 20000, True, False)])
def test_the_faster_one(d, n, k, T, rows, one):
    assert permute_by_hist(d, n, k, T, "bf16", rows) == one


@pytest.mark.gpu
@pytest.mark.parametrize("n,T,k", [c[:3] for c in ROUTE])
def test_permutation_parity(n, T, k):
    inp = make("permute", 32, (32,) * n, T, "bf16", k, seed=31)
    r = _runner(inp)
    r.route()
    check_routing(inp, r.routing_host())


@pytest.mark.gpu
@pytest.mark.parametrize("n,d,T,k,dtype,one", LAYER)
def test_layer_copies_the_right_rows(n, d, T, k, dtype, one):
    inp = make("permute", d, (32,) * n, T, dtype, k, seed=32)
    r = _runner(inp)
    r.route()
    want = {f: getattr(r.routing, f).clone() for f in ("topk_idx", "topk_w", "counts", "offsets", "row_of", "src_of", "near_tie_count")}
    for f in want:
        getattr(r.routing, f).fill_(-7)
    r.fwd()
    for f, w in want.items():
        assert torch.equal(getattr(r.routing, f), w), f
    x, W1, W3, W2 = r.x.float(), r.W1.float().view(n, 32, d), r.W3.float().view(n, 32, d), r.W2.float().view(n, d, 32)
    y = torch.zeros_like(x)
    for e in range(n):
        t, slot = (r.routing.topk_idx.view(T, k) == e).nonzero(as_tuple=True)
        h = torch.nn.functional.silu(x[t] @ W1[e].T) * (x[t] @ W3[e].T)
        y[t] += r.routing.topk_w.view(T, k)[t, slot, None] * (h @ W2[e].T)
    # largest error over the largest output, as in the parity tests: 1e-4 in float32, 2e-2 in bf16
    assert float((r.y.float() - y).abs().max() / y.abs().max()) <= (1e-4 if dtype == "f32" else 2e-2)
