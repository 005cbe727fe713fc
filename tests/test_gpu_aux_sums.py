"""Sums of the gate extensions over many tokens: the means of the auxiliary loss, the gradient of the noise term's gain."""
import pytest
import torch

import paper_2409_12210_amd as m
from choice_probe import choice

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,N", [(1 << 20, 64), (1 << 20, 33), (131073, 64), (8191, 8), (3, 2)])
def test_means_are_rounded_once(T, N):
    """P and f against float64 means of the library's own p and choices.  float32 rounding is 2^-24 = 6e-8, so a mean that is
    rounded once is within that of it; the tolerance leaves a second rounding's room (float32 sums of 2^20 tokens and 64
    experts were off by 7e-7).  The loss adds N products of two such means in float64: the same bound."""
    d, k = 32, 2
    gen = torch.Generator(device="cuda").manual_seed(T + N)
    x = torch.randn((T, d), generator=gen, device="cuda").bfloat16()
    Wg = (0.2 * torch.randn((d, N), generator=gen, device="cuda")).bfloat16()
    f32 = dict(dtype=torch.float32, device="cuda")
    ext = m.GateExt(aux_alpha=0.01, probs=torch.empty((T, N), **f32), aux_f=torch.empty(N, **f32),
                    aux_P=torch.empty(N, **f32), aux_loss=torch.empty(1, **f32))
    r = m.Routing.empty(T, N, k)
    layer = (d, [32] * N, k, "bf16", T)
    ws = torch.empty(m.modse_workspace_size(*layer, m.WS_FWD), dtype=torch.uint8, device="cuda")
    m.modse_route_ext(*layer, x, Wg, None, ext, r, ws)
    torch.cuda.synchronize()
    P = ext.probs.cpu().double().mean(0)
    f = torch.bincount(r.topk_idx[:, 0].cpu(), minlength=N).double() / T
    assert ((ext.aux_P.cpu().double() - P).abs() / P).max() <= 1.2e-7
    assert (ext.aux_f.cpu().double() - f).abs().max() <= 6e-8
    loss = float(torch.tensor(0.01)) * N * float((f * P).sum())
    assert abs(float(ext.aux_loss) - loss) <= 1.2e-7 * loss


def test_dgamma_of_many_equal_tokens():
    """2^20 copies of one token: their shares of dgamma are equal, and the 64 that a wave adds up make a sum without rounding.
    2^14 copies give four float64 sums of 64 such sums each, all of them exact, so that dgamma of 2^20 copies is 64 times theirs.
    Four float32 partial sums are rounded and added: 3 * 2^-24 = 1.8e-7.  (A share's own last bit goes by the order of the
    GEMMs' sums, which a tile shape may change: both batches take the same ones.)"""
    d, d_ff = 32, [32, 32]
    assert len({tuple(choice(g, d, d_ff, 2, T, "f32").bm == 32 for g in ("up", "down", "dh", "dx")) for T in (1 << 14, 1 << 20)}) == 1
    gen = torch.Generator(device="cuda").manual_seed(3)

    def normal(*shape, sigma=1.0):
        return sigma * torch.randn(shape, generator=gen, device="cuda")

    x1, dy1, Wg, Wn = normal(1, d), normal(1, d), normal(d, 2), normal(d, 2)
    W1, W3, W2 = normal(64, d), normal(64, d), normal(64 * d)
    got = []
    for T in (1 << 14, 1 << 20):
        layer = (d, d_ff, 2, "f32", T)
        x, dY, y, dX = x1.repeat(T, 1), dy1.repeat(T, 1), torch.empty((T, d), device="cuda"), torch.empty((T, d), device="cuda")
        ext = m.GateExt(W_noise=Wn, gamma=torch.ones(1, device="cuda"), eps=1e-6, noise_pre=torch.empty((T, 2), device="cuda"))
        r = m.Routing.empty(T, 2, 2)
        saved = torch.empty(m.modse_saved_size(*layer), dtype=torch.uint8, device="cuda")
        ws = torch.empty(max(m.modse_workspace_size(*layer, w) for w in (m.WS_FWD_SAVED, m.WS_BWD)), dtype=torch.uint8,
                         device="cuda")
        g = [torch.empty(n, device="cuda") for n in (2 * d, 2 * d, 1, 64 * d, 64 * d, 64 * d)]
        m.modse_layer_fwd_ext(*layer, x, Wg, None, ext, W1, W3, W2, y, r, saved, ws)
        m.modse_layer_bwd_ext(*layer, x, Wg, ext, 0.0, W1, W3, W2, r, saved, dY, dX, *g, False, ws)
        torch.cuda.synchronize()
        got.append(float(g[2]) / T)
    assert got[0] != 0.0
    assert abs(got[1] - got[0]) <= 1.8e-7 * abs(got[0])
