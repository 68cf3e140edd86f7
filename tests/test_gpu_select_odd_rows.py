"""Selection on rows of odd capacity (a row then starts on any multiple of 4 bytes) and of the lengths at which the
selection changes its way of holding a row: bit-exact against the oracle's selection on the same fp32 scores."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cap,k", [(3, 16381, 700), (2, 33793, 1500), (4, 33795, 2000), (5, 61003, 2048), (2, 65537, 300),
                                        (300, 4099, 200), (300, 14337, 700), (2, 135171, 4000),
                                        # only the larger sample leaves room for them in the lists, or is sure enough
                                        (3, 101388, 12163), (2, 65537, 12000)])
def test_odd_capacities(oracle, rows, cap, k):
    import torch
    from paper_2507_03153_amd import hgca
    rng = np.random.default_rng(cap + rows)
    scores = (rng.standard_normal((1, rows, cap)) + 2.5 * (rng.random((1, rows, cap)) < 0.01)).astype(np.float32)
    scores[0, 0] = np.round(scores[0, 0] * 8) / 8                # ties everywhere in one row
    shape = hgca.Shape(hgca.F32, 1, rows, rows, 128, 1.0)
    d = torch.from_numpy(scores).cuda()
    idx = torch.full((1, rows, k), -7, dtype=torch.int32, device="cuda")
    cnt, sel = torch.zeros(1, rows, dtype=torch.int32, device="cuda"), torch.zeros(1, rows, k, device="cuda")
    hgca.select_topk(shape, d, None, cap, k, k, idx, cnt, sel_scores_out=sel)
    torch.cuda.synchronize()
    want, want_cnt = oracle.select_given(scores, k, k)
    assert np.array_equal(cnt.cpu().numpy(), want_cnt) and np.array_equal(idx.cpu().numpy(), want)
    assert np.array_equal(sel.cpu().numpy(), np.take_along_axis(scores, want.astype(np.int64), axis=2))


@pytest.mark.parametrize("cap", [1021, 2054, 131])
def test_scores_of_odd_capacities(oracle, cap):
    """The score pass writes whole rows of an odd capacity: every score, nothing behind them."""
    import torch
    from paper_2507_03153_amd import hgca
    B, Hq, Hkv, d = 2, 8, 2, 128
    g = torch.Generator().manual_seed(cap)
    q = torch.randn(B, Hq, d, generator=g).to(torch.bfloat16)
    k = torch.randn(B, Hkv, cap, d, generator=g).to(torch.bfloat16)
    shape = hgca.Shape(hgca.BF16, B, Hq, Hkv, d, d ** -0.5)
    out = torch.full((B * Hq * cap + 64,), -9.0, device="cuda")
    hgca.pool_scores(shape, q.cuda(), hgca.Tier(k.cuda(), None, cap), out)
    torch.cuda.synchronize()
    want = torch.einsum("bghd,bgtd->bght", q.double().view(B, Hkv, Hq // Hkv, d), k.double()) * d ** -0.5
    got = out.cpu()
    assert torch.all(got[B * Hq * cap:] == -9.0)
    assert float((got[:B * Hq * cap].double().view(B, Hkv, Hq // Hkv, cap) - want).abs().max()) <= 1e-5


@pytest.mark.parametrize("cap,k", [(33800, 1500), (40000, 1024), (61003, 2048), (65536, 3000), (70001, 2500), (135100, 4000)])
def test_high_scores_that_stand_together(oracle, cap, k):
    """Rows whose high scores are not spread by chance, which the sampled pre-filter leaves to the mode that holds a row as
    bytes: in groups of 8, 64 and 512 consecutive positions, rising towards the end, all at the end, one far above a flat
    row, two levels, and infinite ones among them."""
    import torch
    from paper_2507_03153_amd import hgca
    rng = np.random.default_rng(cap)
    pos = np.arange(cap)
    rows = [rng.standard_normal(cap) + 5.0 * np.repeat(rng.random(-(-cap // g)) < 1.2 * k / cap, g)[:cap] for g in (8, 64, 512)]
    rows += [rng.standard_normal(cap) + 6.0 * pos / cap, rng.standard_normal(cap) - 4.0 * np.log(cap - pos)]
    rows += [np.where(pos == 5, 1e6, rng.standard_normal(cap)), np.where(pos // 700 % 5 == 0, 1.0, 0.0)]
    rows += [np.where(pos % 9001 < 40, np.inf, rng.standard_normal(cap)), np.where(pos < cap // 2, -np.inf, rng.standard_normal(cap))]
    scores = np.stack(rows).astype(np.float32)[None]
    n = scores.shape[1]
    shape = hgca.Shape(hgca.F32, 1, n, n, 128, 1.0)
    idx = torch.full((1, n, k), -7, dtype=torch.int32, device="cuda")
    cnt, sel = torch.zeros(1, n, dtype=torch.int32, device="cuda"), torch.zeros(1, n, k, device="cuda")
    hgca.select_topk(shape, torch.from_numpy(scores).cuda(), None, cap, k, k, idx, cnt, sel_scores_out=sel)
    torch.cuda.synchronize()
    want, want_cnt = oracle.select_given(scores, k, k)
    assert np.array_equal(cnt.cpu().numpy(), want_cnt)
    for r in range(n):
        assert np.array_equal(idx.cpu().numpy()[0, r], want[0, r]), r
    assert np.array_equal(sel.cpu().numpy(), np.take_along_axis(scores, want.astype(np.int64), axis=2))
