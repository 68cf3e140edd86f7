"""Query-averaged weights for heads of 64, whose pass works row tiles off two at a time in groups of up to 4: every count of row
tiles and one more block, over one tier and over two, against softmax in 64 bits.  Bar: 2e-5 absolute (weights are at most 1; exact
products, sums and exponentials in fp32, as for the window's weights)."""
import pytest

pytestmark = pytest.mark.gpu


def reference(torch, q, k, scale, n_seen):
    """Weights [B, Hq, T] averaged over the queries, and the lse [B, N, Hq]; n_seen[i]: tokens that query i sees."""
    B, N, Hq, d = q.shape
    Hkv, T = k.shape[1], k.shape[2]
    s = (q.double().view(B, N, Hkv, Hq // Hkv, 1, d) * k.double().view(B, 1, Hkv, 1, T, d)).sum(-1).view(B, N, Hq, T) * scale
    s = s.masked_fill(torch.arange(T, device=q.device).view(1, 1, 1, T) >= n_seen.view(1, N, 1, 1), float("-inf"))
    lse = torch.logsumexp(s, -1)
    return torch.exp(s - lse[..., None]).mean(1), lse


@pytest.mark.parametrize("group", [1, 2, 4, 8])
@pytest.mark.parametrize("rows", [8, 40, 72, 104, 128, 136])
def test_heads_of_64(group, rows):
    import torch
    from paper_2507_03153_amd import hgca
    B, Hkv, d, W, P, dev = 1, 2, 64, 700, 2900, "cuda:0"
    N = rows // group
    g = torch.Generator(device=dev).manual_seed(rows + group)
    q = torch.randn(B, N, Hkv * group, d, generator=g, device=dev).bfloat16()
    kw, kp = (torch.randn(B, Hkv, n, d, generator=g, device=dev).bfloat16() for n in (W, P))
    scale, shape = d ** -0.5, hgca.Shape(hgca.BF16, B, Hkv * group, Hkv, d, d ** -0.5)
    seen = W - N + 1 + torch.arange(N, device=dev)               # the queries are the window's last tokens
    a_w, lse_w = reference(torch, q, kw, scale, seen)
    a_p, lse_p = reference(torch, q, kp, scale, torch.full((N,), P, device=dev))
    lw, lp = lse_w.float().contiguous(), lse_p.float().contiguous()
    tw, tp = hgca.Tier(kw, None, W), hgca.Tier(kp, None, P)
    f32 = dict(dtype=torch.float32, device=dev)
    one_w, one_p, two_w, two_p = (torch.full((B, Hkv * group, n), -1.0, **f32) for n in (W, P, W, P))
    hgca.append_weights(shape, q, tw, True, lw, one_w)
    hgca.append_weights(shape, q, tp, False, lp, one_p)
    hgca.append_weights_tiers(shape, q, tw, tp, lw, lp, two_w, two_p)
    torch.cuda.synchronize()
    for got, want in ((one_w, a_w), (one_p, a_p), (two_w, a_w), (two_p, a_p)):
        assert float((got.double() - want).abs().max()) <= 2e-5
