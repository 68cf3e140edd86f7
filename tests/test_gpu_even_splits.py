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


# The host's split sizes (multiples of 64, at least 64 and at most 512) and the kernels' evening of them, mirrored: the
# cases below are of use only where the host's size is above what the kernels leave alone, 16 384 / head_dim tokens.
def host_chunk(cap, units, target):
    want = max(1, target // units)
    return min(512, max(64, (-(-cap // want) + 63) // 64 * 64))


def evened(chunk, n, n_splits, d):
    if chunk <= 16384 // d or n > chunk * (n_splits - 1):
        return chunk
    return min(chunk, max((-(-n // n_splits) + 63) // 64 * 64, 16384 // d))


def parts_in_use(ws, rows, d, cap, n_splits):
    """Per row, the number of splits that hold something, from the partial maxima that a call leaves in its workspace."""
    import torch
    at = (rows * -(-cap // 64) * d * 4 + 255) // 256 * 256
    m = ws[at:at + rows * n_splits * 4].view(torch.float32).view(rows, n_splits)
    return (m > float("-inf")).sum(1).cpu().numpy()


@pytest.mark.parametrize("name,kw", [
    ("C2", dict(Hq=16, Hkv=4)), ("C2", dict(Hq=16, Hkv=16, d=64)), ("C2", dict(Hq=32, Hkv=4)), ("C1", dict(Hq=16, Hkv=4, d=128)),
], ids=["gqa4", "mha_d64", "gqa8_two_launches", "fp32"])
def test_lists_and_windows_whose_splits_are_evened(oracle, name, kw):
    import torch
    from paper_2507_03153_amd import hgca, runner
    W, k_max = 8192, 8192
    w_lens = [8192, 7681, 7680, 4096, 4097, 2049, 2048, 1500, 129, 128, 1, 0]
    counts = [0, 1, 127, 128, 129, 2047, 2048, 2049, 4097, 4096, 7680, 8192]
    B = len(w_lens)
    cfg = wl.scaled(wl.CONFIGS[name], B=B, W=W, P=9000, k=16, ragged=None, **kw)
    fp32 = cfg.dtype == "f32"
    two_launches = fp32 or cfg.Hq // cfg.Hkv == 8
    chunk_w = host_chunk(W, B * cfg.Hkv, 1024 if two_launches else 512)
    chunk_l = host_chunk(k_max, B * cfg.Hq, 2048)
    n_w, n_l = -(-W // chunk_w), -(-k_max // chunk_l)
    assert chunk_w > 16384 // cfg.d and chunk_l > 16384 // cfg.d                # else nothing is evened
    assert len({evened(chunk_w, n, n_w, cfg.d) for n in w_lens}) > 2 and len({evened(chunk_l, n, n_l, cfg.d) for n in counts}) > 2
    L = wl.make_layer(cfg)
    L.window.seq_lens = np.array(w_lens, np.int32)
    rng = np.random.default_rng(7)
    idx = np.full((B, cfg.Hq, k_max), -1, np.int32)
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
    rows = B * cfg.Hq
    for ws, cap, chunk, lens in ((step.ws_dense, W, chunk_w, w_lens), (step.ws_sparse, k_max, chunk_l, counts)):
        n_splits = -(-cap // chunk)
        want = [-(-n // evened(chunk, n, n_splits, cfg.d)) for n in lens]
        assert np.array_equal(parts_in_use(ws, rows, cfg.d, cap, n_splits).reshape(B, cfg.Hq), np.repeat(np.array(want)[:, None], cfg.Hq, 1))
    tier = lambda t: oracle.Tier(t.k, t.v, t.cap, t.seq_lens, t.block_table, t.block_size)
    o, lse = oracle.attend_union(L.q, tier(L.window), tier(L.pool), idx, cnt, L.scale)
    tol = 1e-5 if fp32 else 2e-4
    assert np.max(np.abs(step.o.double().cpu().numpy() - o)) <= tol
    assert np.max(np.abs(step.lse.double().cpu().numpy() - lse)) <= tol


def test_a_token_joins_a_window_whose_splits_are_evened():
    """The managed decode step in one call: the split that owns the new token's position, which follows from the grown
    length, writes its rows.  Windows a third to a half full, lengths that cross the ends of evened splits and the lengths at
    which the splits grow (2048 = 16 splits of 128)."""
    import torch
    from paper_2507_03153_amd import cache, hgca, runner
    from test_gpu_kv_manager import run_loop
    hgca.lib()
    B, Hq, Hkv, d, W = 4, 16, 8, 128, 4096
    prefill, steps = (1276, 2043, 2047, 1919), 8
    chunk = host_chunk(W, B * Hkv, 512)
    assert chunk > 16384 // d and all(evened(chunk, p + 1, W // chunk, d) < chunk for p in prefill)
    assert evened(chunk, 2048, W // chunk, d) != evened(chunk, 2049, W // chunk, d)
    C, _, status = run_loop((torch, hgca, runner, cache), B=B, Hq=Hq, Hkv=Hkv, d=d, block_size=16, win_blocks=W // 16,
                            max_blocks=W // 16 + 2, k_max=64, prefill=prefill, steps=steps, alpha=0.3, beta=1.0, seed=17, one_call=True)
    assert status == 0 and C.win_lens.cpu().tolist() == [p + steps for p in prefill]
    want = [-(-(p + steps) // evened(chunk, p + steps, W // chunk, d)) for p in prefill]
    assert np.array_equal(parts_in_use(C.ws_dense, B * Hq, d, W, W // chunk).reshape(B, Hq), np.repeat(np.array(want)[:, None], Hq, 1))
