"""Append-stage attention over pool and window as one line of tokens: lengths at which the shares of the line fall on,
before and behind the boundary between the tiers, several blocks of query rows, and paged tiers whose block size is no
power of two."""
import numpy as np
import pytest

from test_gpu_append import gpu, make_inputs, run_case, to_paged  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(B=3, N=9, Hq=8, Hkv=2, d=128, W=128, P=1024, w_lens=(128, 9, 64), p_lens=(1024, 1000, 0)),   # whole steps, no pool
    dict(B=1, N=70, Hq=16, Hkv=2, d=128, W=200, P=700),                      # five row blocks, streams no multiple of 8
    dict(B=1, N=4, Hq=4, Hkv=1, d=128, W=640, P=5000),                       # more shares than a unit has elsewhere
    dict(B=2, N=33, Hq=2, Hkv=2, d=64, W=65, P=4033, w_lens=(65, 33), p_lens=(1, 4033)),
    dict(B=9, N=130, Hq=4, Hkv=1, d=64, W=192, P=320, w_lens=(192, 130, 131, 160, 191, 150, 140, 170, 180),
         p_lens=(320, 0, 64, 63, 65, 128, 1, 319, 256)),
], ids=["boundaries", "row_blocks", "many_shares", "d64_ragged", "ragged_row_blocks"])
def test_shares_of_the_line(gpu, kw):  # noqa: F811
    run_case(gpu, 71, **kw)


@pytest.mark.parametrize("block", [16, 48, 80, 64])
def test_block_sizes_read_the_same_rows(gpu, block):  # noqa: F811
    """The same rows in blocks of any size: bit-identical to the contiguous tier (same arithmetic, same shares)."""
    torch, hgca, runner = gpu
    B, N, Hq, Hkv, d, W, P = 2, 40, 8, 2, 128, 240, 1200
    q, Kw, Vw, wl_, Kp, Vp, pl_ = make_inputs(5, B, N, Hq, Hkv, d, W, P, (240, 77), (1200, 611))
    g = lambda a: runner._to_gpu(a, "cuda:0")
    shape = hgca.Shape(hgca.BF16, B, Hq, Hkv, d, 1.0 / np.sqrt(d))
    tiers = [(hgca.Tier(g(Kw), g(Vw), W, g(wl_)), hgca.Tier(g(Kp), g(Vp), P, g(pl_))),
             (to_paged(runner, hgca, torch, Kw, Vw, wl_, W, block, 1, "cuda:0"),
              to_paged(runner, hgca, torch, Kp, Vp, pl_, P, block, 2, "cuda:0"))]
    out = []
    for win, pool in tiers:
        f = lambda *s: torch.full(s, float("nan"), dtype=torch.float32, device="cuda:0")
        o, lse, lw, lp, a_w, a_p = f(B, N, Hq, d), f(B, N, Hq), f(B, N, Hq), f(B, N, Hq), f(B, Hq, W), f(B, Hq, P)
        ws = hgca.append_tiers_workspace(shape, N, W, P, "cuda:0")
        hgca.append_attn_tiers(shape, g(q), win, pool, o, lse, ws, lse_window_out=lw, lse_pool_out=lp)
        hgca.append_weights_tiers(shape, g(q), win, pool, lw, lp, a_w, a_p)
        out.append((o, lse, lw, lp, a_w, a_p))
    torch.cuda.synchronize()
    for x, y in zip(*out):
        assert torch.isfinite(x).all() and torch.equal(x, y)


def test_one_part_repeats_itself(gpu):  # noqa: F811
    """Weights rounded once to bf16: O depends on how the line is cut (a weight is rounded relative to the maximum of its
    share), and on nothing else: the same call gives the same bits, into a workspace that held something else."""
    torch, hgca, runner = gpu
    B, N, Hq, Hkv, d, W, P, dev = 2, 48, 64, 8, 128, 1024, 7000, "cuda:0"
    g = torch.Generator(device=dev).manual_seed(8)
    r = lambda *s: torch.randn(*s, generator=g, device=dev).to(torch.bfloat16)
    q, win, pool = r(B, N, Hq, d), hgca.Tier(r(B, Hkv, W, d), r(B, Hkv, W, d), W), hgca.Tier(r(B, Hkv, P, d), r(B, Hkv, P, d), P)
    shape = hgca.Shape(hgca.BF16, B, Hq, Hkv, d, d ** -0.5)
    out = []
    for fill in (0, 255):
        o, lse = torch.zeros(B, N, Hq, d, device=dev), torch.zeros(B, N, Hq, device=dev)
        ws = hgca.append_tiers_workspace(shape, N, W, P, dev).fill_(fill)
        hgca.append_attn_tiers(shape, q, win, pool, o, lse, ws, one_part_p=True)
        out.append((o, lse))
    torch.cuda.synchronize()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("B,Hq,Hkv,N,W,P,shares", [
    (1, 32, 8, 64, 1000, 7000, 16),                              # 16 units: one workgroup per compute unit
    (2, 4, 4, 55, 836, 4759, 30),                                # 8 units, 89 steps in threes
    (2, 4, 4, 100, 512, 5632, 32),
    (8, 32, 8, 32, 4096, 28672, 8),                              # 64 units, long shares: two workgroups per compute unit
    (2, 32, 8, 509, 4096, 28672, 2),
], ids=["n64", "n55", "n100", "n32", "n509"])
def test_number_of_shares(gpu, B, Hq, Hkv, N, W, P, shares):  # noqa: F811
    """The number of shares a call is cut into, as the partials in its workspace show it: shares + 1 slots of a row of
    outputs and two statistics per (sequence, query, head), every one of them written."""
    torch, hgca, runner = gpu
    d, dev = 128, "cuda:0"
    z = lambda *s: torch.zeros(*s, dtype=torch.bfloat16, device=dev)
    shape = hgca.Shape(hgca.BF16, B, Hq, Hkv, d, 1.0)
    o, lse = torch.zeros(B, N, Hq, d, device=dev), torch.zeros(B, N, Hq, device=dev)
    ws = hgca.append_tiers_workspace(shape, N, W, P, dev).fill_(255)             # NaN everywhere
    win, pool = hgca.Tier(z(B, Hkv, W, d), z(B, Hkv, W, d), W), hgca.Tier(z(B, Hkv, P, d), z(B, Hkv, P, d), P)
    hgca.append_attn_tiers(shape, z(B, N, Hq, d), win, pool, o, lse, ws)
    torch.cuda.synchronize()
    written = int((~torch.isnan(ws.view(torch.float32))).sum())
    assert written == B * N * Hq * (shares + 1) * (d + 2)
