"""Splits of a window or a salient list that fill only part of their capacity: the number of splits follows the
capacity, the tokens per split follow the actual length, so every edge between full, short and empty splits is a
length of its own here.  Bars as in test_gpu_parity: fp32 accumulation over exact products."""
import numpy as np
import pytest

from paper_2507_03153_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,kw", [
    ("C2", dict(Hq=8, Hkv=2)), ("C2", dict(Hq=4, Hkv=4, d=64)), ("C2", dict(Hq=16, Hkv=2)), ("C1", dict(Hq=8, Hkv=2)),
], ids=["gqa4", "mha_d64", "gqa8_two_launches", "fp32"])
def test_lists_and_windows_shorter_than_their_capacity(oracle, name, kw):
    import torch
    from paper_2507_03153_amd import hgca, runner
    w_lens = [0, 1, 63, 64, 65, 300, 1024]
    counts = [2048, 513, 65, 64, 63, 1, 0]
    cfg = wl.scaled(wl.CONFIGS[name], B=len(counts), W=1024, P=2500, k=16, ragged=None, **kw)
    L = wl.make_layer(cfg)
    L.window.seq_lens = np.array(w_lens, np.int32)
    rng = np.random.default_rng(7)
    k_max = max(counts)
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
    assert np.max(np.abs(step.o.double().cpu().numpy() - o)) <= tol
    assert np.max(np.abs(step.lse.double().cpu().numpy() - lse)) <= tol
