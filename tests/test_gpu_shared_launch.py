"""Steps whose window splits and gather share a launch in fp32 and in groups of 8, on both sides of the rule for those groups:
steady steps against the oracle, and the one-call managed step, where the split that owns the token's position inserts it,
against the same step as separate calls (which insert it first), over block boundaries and evictions.  Bars as in
test_gpu_parity; the two managed loops differ by the order of fp32 sums only."""
import numpy as np
import pytest

from paper_2507_03153_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,kw,k_max", [
    ("C1", dict(Hq=4, Hkv=4), 130), ("C1", dict(Hq=4, Hkv=2, d=128), 513), ("C1", dict(Hq=16, Hkv=2, block_size=16), 64),
    ("C2", dict(Hq=16, Hkv=2), 150), ("C2", dict(Hq=64, Hkv=8), 700), ("C2", dict(Hq=16, Hkv=2, d=64, block_size=32), 257),
], ids=["fp32_mha", "fp32_gqa2_d128", "fp32_gqa8_paged", "gqa8", "gqa8_two_launches", "gqa8_d64_paged"])
def test_steady_step(oracle, name, kw, k_max):
    import torch
    from paper_2507_03153_amd import hgca, runner
    w_lens, counts = [0, 1, 257, 600], [k_max, 0, 1, k_max - 1]
    cfg = wl.scaled(wl.CONFIGS[name], B=len(counts), W=600, P=900, k=16, ragged=None, **kw)
    L = wl.make_layer(cfg)
    L.window.seq_lens = np.array(w_lens, np.int32)
    rng = np.random.default_rng(11)
    idx = np.full((cfg.B, cfg.Hq, k_max), -1, np.int32)
    for b, c in enumerate(counts):
        for h in range(cfg.Hq):
            idx[b, h, :c] = np.sort(rng.choice(cfg.P, c, replace=False))
    cnt = np.repeat(np.array(counts, np.int32)[:, None], cfg.Hq, axis=1)
    D = runner.DeviceLayer.upload(L)
    step = runner.HybridStep(D.shape, cfg.W, cfg.P, k_max)
    step.idx.copy_(torch.from_numpy(idx))
    step.cnt.copy_(torch.from_numpy(cnt))
    hgca.hybrid_decode_step_selected(D.shape, D.q, D.window, D.pool, step.idx, step.cnt, k_max, step.o, step.lse,
                                     step.ws_dense, step.ws_sparse)
    torch.cuda.synchronize()
    tier = lambda t: oracle.Tier(t.k, t.v, t.cap, t.seq_lens, t.block_table, t.block_size)
    o, lse = oracle.attend_union(L.q, tier(L.window), tier(L.pool), idx, cnt, L.scale)
    tol = 1e-5 if cfg.dtype == "f32" else 2e-4
    got_l = step.lse.double().cpu().numpy()
    assert np.array_equal(np.isinf(got_l), np.isinf(lse))
    some = np.isfinite(lse)
    assert np.max(np.abs(step.o.double().cpu().numpy() - o)) <= tol
    assert np.max(np.abs(got_l[some] - lse[some])) <= tol


@pytest.mark.parametrize("dtype,Hq,Hkv,d,k_max", [
    ("f32", 4, 4, 64, 64), ("f32", 8, 2, 128, 40), ("f32", 8, 1, 64, 300), ("bf16", 16, 2, 128, 64), ("bf16", 16, 2, 64, 64),
    ("bf16", 64, 8, 128, 1024),
], ids=["fp32_mha", "fp32_gqa4_d128", "fp32_gqa8", "gqa8", "gqa8_d64", "gqa8_two_launches"])
def test_managed_step_equals_separate_calls(dtype, Hq, Hkv, d, k_max):
    import torch
    from paper_2507_03153_amd import cache
    dev, dt = "cuda:0", torch.float32 if dtype == "f32" else torch.bfloat16
    B, bs, wb, steps, alpha, beta = 3, 16, 2, 40, 0.3, 1.0
    g = torch.Generator(device=dev).manual_seed(5)
    C = [cache.LayerCache(dt, B, Hq, Hkv, d, bs, wb, 8, k_max, d ** -0.5, dev) for _ in range(2)]
    for t in range(steps):
        q = torch.randn(B, Hq, d, generator=g, device=dev).to(dt)
        k, v = (torch.randn(B, Hkv, d, generator=g, device=dev).to(dt) for _ in range(2))
        for c, one_call in zip(C, (True, False)):
            c.decode_step(q, k, v, alpha, beta, one_call=one_call)
        torch.cuda.synchronize()
        tol = 1e-5 if dtype == "f32" else 2e-4
        assert float((C[0].o - C[1].o).abs().max()) <= tol and float((C[0].lse - C[1].lse).abs().max()) <= tol, t
        assert torch.equal(C[0].win_lens, C[1].win_lens) and torch.equal(C[0].pool_lens, C[1].pool_lens)
        assert torch.equal(C[0].ctx_cnt, C[1].ctx_cnt) and torch.equal(C[0].ctx_idx, C[1].ctx_idx), t
        assert float((C[0].a_maw - C[1].a_maw).abs().max()) <= 2e-5
    assert torch.equal(C[0].k_blocks, C[1].k_blocks) and torch.equal(C[0].v_blocks, C[1].v_blocks)
    assert int(C[0].pool_lens.min()) > 0 and int(C[0].status.cpu()[0]) == int(C[1].status.cpu()[0])
