"""The auxiliary loss over many tokens and experts: one block sums all probabilities, so its sums are long."""
import pytest
import torch

import paper_2409_12210_amd as m

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
