"""Append attention with a large offset common to all scores: rows whose maximum stands must not drift while other rows
of their wave find new maxima, hundreds of times over a long tier."""
import pytest

from test_gpu_append import gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("one_part", [False, True], ids=["two_parts", "one_part"])
@pytest.mark.parametrize("offset", [10.0, 60.0])
def test_lse_of_scores_with_a_common_offset(gpu, offset, one_part):  # noqa: F811
    torch, hgca, runner = gpu
    dev = "cuda:0"
    B, N, H, d, P = 8, 32, 64, 64, 8192                          # 512 units: one workgroup walks all 128 steps
    g = torch.Generator(device=dev).manual_seed(5)
    u = torch.nn.functional.normalize(torch.randn(B, H, 1, d, generator=g, device=dev), dim=-1)
    q = (torch.randn(B, H, N, d, generator=g, device=dev) + 8 * u).to(torch.bfloat16)
    k = (torch.randn(B, H, P, d, generator=g, device=dev) + offset * d ** 0.5 / 8 * u).to(torch.bfloat16)
    v = torch.randn(B, H, P, d, generator=g, device=dev, dtype=torch.bfloat16)
    shape = hgca.Shape(hgca.BF16, B, H, H, d, d ** -0.5)
    qn = q.transpose(1, 2).contiguous()
    o, lse = torch.zeros(B, N, H, d, device=dev), torch.zeros(B, N, H, device=dev)
    hgca.append_attn(shape, qn, hgca.Tier(k, v, P), False, o, lse, hgca.append_workspace(shape, N, P, dev), one_part_p=one_part)
    torch.cuda.synchronize()
    err = top = 0.0
    for b in range(B):
        s = torch.bmm(q[b].double(), k[b].double().transpose(1, 2).contiguous()) * d ** -0.5
        err = max(err, float((lse[b].double().transpose(0, 1) - s.logsumexp(-1)).abs().max()))
        top = max(top, float(s.abs().max()))
    # the weights' sum as for small scores (5e-6), and four roundings to 2^-24 of the largest score: the score's own sum,
    # its product with the scale, the shift, lse
    bar = 5e-6 + 4 * top * 2.0 ** -24
    print(f"\n[case] offset {offset}: largest score {top:.1f}, max|dlse|={err:.2e} (bar {bar:.2e})", flush=True)
    assert err <= bar
