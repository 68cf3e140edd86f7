"""Query-averaged weights at the row counts and lengths where the pass changes its way: row tiles that exist in part, tiles
dealt out to waves that have no tokens of their own, several passes over the rows of one block of tokens."""
import pytest

from test_gpu_append import gpu, run_case, run_case_f32  # noqa: F401

pytestmark = pytest.mark.gpu

EDGES = [
    dict(B=2, N=31, Hq=4, Hkv=1, d=128, W=100, P=700),                       # 124 rows: the last tile in part
    dict(B=1, N=33, Hq=8, Hkv=2, d=128, W=64, P=300),                        # 132 rows: a second block of four rows
    dict(B=1, N=24, Hq=8, Hkv=2, d=128, W=96, P=2000, p_lens=(1999,)),       # three tiles
    dict(B=3, N=9, Hq=8, Hkv=1, d=64, W=70, P=64, w_lens=(70, 9, 4)),        # shares of one step, a prompt longer than the window
    dict(B=2, N=100, Hq=2, Hkv=2, d=64, W=128, P=33),                        # four tiles on shares of one step
    dict(B=1, N=1, Hq=2, Hkv=2, d=128, W=1, P=130),
]
IDS = ["rows124", "rows132", "rows96", "rows72", "rows100", "row1"]


@pytest.mark.parametrize("kw", EDGES, ids=IDS)
def test_edges_bf16(gpu, kw):  # noqa: F811
    run_case(gpu, 61, **kw)


@pytest.mark.parametrize("kw", EDGES, ids=IDS)
def test_edges_fp32(gpu, kw):  # noqa: F811
    run_case_f32(gpu, 62, **kw)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_long_shares_with_several_blocks_of_rows(gpu, dtype):  # noqa: F811
    """256 (sequence, head) pairs, so a share is a whole row of tokens: it goes through blocks of 2048 of them, each once
    per 128 rows.  A key that is not finite touches its own token only."""
    torch, hgca, runner = gpu
    B, H, N, d, P, dev = 32, 8, 140, 64, 2300, "cuda:0"
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device=dev).manual_seed(9)
    q, k = (torch.randn(*s, generator=g, device=dev).to(dt) for s in ((B, N, H, d), (B, H, P, d)))
    lens = torch.full((B,), P, dtype=torch.int32, device=dev)
    lens[1], lens[2] = 2049, 77                                  # one shorter than the prompt
    shape = hgca.Shape(hgca.BF16 if dtype == "bf16" else hgca.F32, B, H, H, d, d ** -0.5)
    tok = torch.arange(P, device=dev)
    for causal in (True, False):
        want, lse = torch.zeros(B, H, P, dtype=torch.float64, device=dev), torch.zeros(B, N, H, device=dev)
        for b in range(B):
            s = torch.matmul(q[b].double().transpose(0, 1).contiguous(), k[b].double().transpose(1, 2).contiguous()) * d ** -0.5
            last = lens[b] - N + torch.arange(N, device=dev) + 1 if causal else lens[b].expand(N)
            s = s.masked_fill(tok[None, None] >= last[None, :, None], float("-inf"))
            l = s.logsumexp(-1)
            want[b] = torch.where(l[..., None] == float("-inf"), 0.0, (s - l[..., None]).exp()).mean(1)
            lse[b] = l.transpose(0, 1).float()
        a = torch.full((B, H, P), float("nan"), device=dev)
        hgca.append_weights(shape, q, hgca.Tier(k, None, P, lens), causal, lse, a)
        k2 = k.clone()
        k2[:, 3, 70, 1], k2[0, 5, P - 1, 0] = float("inf"), float("nan")
        a2 = torch.full_like(a, float("nan"))
        hgca.append_weights(shape, q, hgca.Tier(k2, None, P, lens), causal, lse, a2)
        torch.cuda.synchronize()
        err = float((a.double() - want).abs().max())
        print(f"\n[case] {dtype} causal={causal}: max|dA|={err:.2e}", flush=True)
        assert err <= (2e-5 if dtype == "bf16" else 1e-5)        # the bars of the append tests
        touched = torch.zeros(B, H, P, dtype=torch.bool, device=dev)
        touched[:, 3, 70], touched[0, 5, P - 1] = True, True
        assert torch.equal(a2[~touched], a[~touched])
