"""Decode steps on each path that a rule may send them to, beside the edge of the rule: every case names the path it is meant for
and asks the rule (csrc/routes.hpp) whether that is where it goes.  Steps with a selection against the oracle's selection and
attention, steps over given lists against the oracle's attention over them.  Bars as in test_gpu_parity."""
import numpy as np
import pytest

from paper_2507_03153_amd import workloads as wl
from routes_rules import rules  # noqa: F401

pytestmark = pytest.mark.gpu

# name, base, heads, sequences, window, pool, k_max, two launches (1) or the general path (0), order of the gather there
STEPS = [
    ("f32_g4_d64", "C1", dict(Hq=32, Hkv=8), 9, 150, 700, 30, 0, 0), ("f32_g4_d64_by_group", "C1", dict(Hq=32, Hkv=8), 9, 150, 700, 120, 0, 1),
    ("f32_g4_d128", "C1", dict(Hq=8, Hkv=2, d=128), 3, 300, 9000, 780, 0, 0),
    ("f32_g4_d128_by_group", "C1", dict(Hq=8, Hkv=2, d=128), 3, 300, 2500, 780, 0, 1),
    ("f32_g8_d64", "C1", dict(Hq=64, Hkv=8), 5, 200, 900, 30, 0, 0), ("f32_g8_d64_by_group", "C1", dict(Hq=64, Hkv=8), 5, 200, 900, 130, 0, 1),
    ("f32_g8_d128", "C1", dict(Hq=16, Hkv=2, d=128), 3, 600, 20000, 780, 0, 0),
    ("f32_g8_d128_by_group", "C1", dict(Hq=16, Hkv=2, d=128), 3, 600, 2000, 780, 0, 1),
    ("f32_g2_d64", "C1", dict(Hq=16, Hkv=8), 17, 500, 800, 100, 0, 0), ("f32_g1_d128", "C1", dict(Hq=40, Hkv=40, d=128), 7, 100, 500, 60, 0, 0),
    ("f32_g8_d64_keys_and_list", "C1", dict(Hq=64, Hkv=8), 1, 100, 33000, 1500, 0, 1),
    ("f32_g8_d64_short", "C1", dict(Hq=64, Hkv=8), 1, 100, 16000, 1500, 1, 1),
    ("bf16_256_rows", "C2", dict(Hq=32, Hkv=8), 8, 100, 700, 40, 1, 0), ("bf16_264_rows", "C2", dict(Hq=24, Hkv=6), 11, 100, 700, 40, 0, 0),
    ("f32_256_rows", "C1", dict(Hq=32, Hkv=8), 8, 100, 700, 40, 1, 0), ("f32_264_rows_one_split_windows", "C1", dict(Hq=33, Hkv=33), 8, 300, 400, 40, 0, 0),
    ("bf16_g8_32_mb", "C2", dict(Hq=16, Hkv=2), 4, 100, 16384, 200, 1, 0), ("bf16_g8_over_32_mb", "C2", dict(Hq=16, Hkv=2), 4, 100, 16400, 200, 0, 0),
    ("bf16_g8_by_group", "C2", dict(Hq=64, Hkv=8), 5, 300, 3000, 150, 0, 1),
]


def layer(name, kw, B, W, P, k_max, ragged):
    cfg = wl.scaled(wl.CONFIGS[name], B=B, W=W, P=P, k=16, ragged=None, **kw)
    L = wl.make_layer(cfg)
    if ragged and B > 1:                         # a full sequence, short ones, empty ones
        rng = np.random.default_rng(B + k_max)
        w, p = rng.integers(0, W + 1, B), rng.integers(0, P + 1, B)
        w[0], p[0], w[1], p[-1] = W, P, 0, 0
        L.window.seq_lens, L.pool.seq_lens = w.astype(np.int32), p.astype(np.int32)
    return cfg, L


def compare(o, lse, want_o, want_lse, tol):
    o, lse = o.double().cpu().numpy(), lse.double().cpu().numpy()
    assert np.array_equal(np.isinf(lse), np.isinf(want_lse))
    some = np.isfinite(want_lse)
    assert np.max(np.abs(o - want_o)) <= tol and np.max(np.abs(lse[some] - want_lse[some])) <= tol


@pytest.mark.parametrize("name,kw,B,W,P,k_max,short,order", [c[1:] for c in STEPS], ids=[c[0] for c in STEPS])
def test_step_with_a_selection(oracle, rules, name, kw, B, W, P, k_max, short, order):
    import torch
    from paper_2507_03153_amd import hgca, runner
    cfg, L = layer(name, kw, B, W, P, k_max, True)
    f32, G = cfg.dtype == "f32", cfg.Hq // cfg.Hkv
    assert rules(f"short {f32:d} {cfg.d} {B * cfg.Hkv} {G} {W} {P} {k_max}", f"order {G} {k_max} {P} 1 0") == [short, order]
    D = runner.DeviceLayer.upload(L)
    step = runner.HybridStep(D.shape, W, P, k_max)
    tier = lambda t: oracle.Tier(t.k, t.v, t.cap, t.seq_lens, t.block_table, t.block_size)
    o, lse, idx, cnt = oracle.hybrid_step(L.q, tier(L.window), tier(L.pool), k_max, k_max, L.scale)
    sel_idx, sel_cnt, sel = torch.empty_like(step.idx), torch.empty_like(step.cnt), torch.zeros_like(step.sel_scores)
    hgca.select_salient(D.shape, D.q, D.pool, k_max, k_max, sel_idx, sel_cnt, step.ws_sparse, sel_scores_out=sel)
    hgca.hybrid_decode_step(D.shape, D.q, D.window, D.pool, k_max, k_max, step.idx, step.cnt, step.o, step.lse, step.ws_dense,
                            step.ws_sparse)
    torch.cuda.synchronize()
    assert torch.equal(step.idx, sel_idx) and np.array_equal(step.cnt.cpu().numpy(), cnt)
    tol = 1e-5 if f32 else 2e-4
    compare(step.o, step.lse, o, lse, tol)
    # the same lists with the selection's scores given, and without
    o2, lse2 = torch.empty_like(step.o), torch.empty_like(step.lse)
    for scores in (sel, None):
        hgca.hybrid_decode_step_selected(D.shape, D.q, D.window, D.pool, sel_idx, sel_cnt, k_max, o2, lse2, step.ws_dense,
                                         step.ws_sparse, sel_scores=scores)
        torch.cuda.synchronize()
        compare(o2, lse2, o, lse, tol)


# name, base, heads, sequences, window, pool, k_max, order of the gather, window first in a shared launch
LISTS = [
    ("bf16_g8_head_by_head", "C2", dict(Hq=64, Hkv=8), 4, 500, 14000, 600, 0, 0), ("bf16_g8_by_group", "C2", dict(Hq=64, Hkv=8), 4, 500, 14000, 700, 1, 0),
    ("bf16_g8_kept", "C2", dict(Hq=64, Hkv=8), 4, 500, 14000, 900, 2, 0), ("bf16_g4_head_by_head", "C2", dict(Hq=32, Hkv=8), 3, 500, 8000, 719, 0, 0),
    ("bf16_g4_kept", "C2", dict(Hq=32, Hkv=8), 3, 500, 8000, 720, 2, 0), ("bf16_g2_by_group", "C2", dict(Hq=16, Hkv=8), 3, 500, 8000, 700, 1, 0),
    ("f32_g1_gather_first", "C1", dict(Hq=8, Hkv=8), 4, 300, 2000, 400, 0, 0), ("f32_g1_window_first", "C1", dict(Hq=8, Hkv=8), 4, 900, 2000, 400, 0, 1),
    ("f32_g2", "C1", dict(Hq=8, Hkv=4), 4, 100, 2000, 600, 1, 1), ("f32_g4_d128", "C1", dict(Hq=16, Hkv=4, d=128), 4, 900, 2000, 100, 0, 1),
    ("f32_g8_kept", "C1", dict(Hq=16, Hkv=2), 4, 700, 2000, 200, 2, 1), ("f32_one_split_windows", "C1", dict(Hq=64, Hkv=32), 9, 500, 400, 30, 0, 1),
]


@pytest.mark.parametrize("name,kw,B,W,P,k_max,order,first", [c[1:] for c in LISTS], ids=[c[0] for c in LISTS])
def test_step_over_given_lists(oracle, rules, name, kw, B, W, P, k_max, order, first):
    import torch
    from paper_2507_03153_amd import hgca, runner
    cfg, L = layer(name, kw, B, W, P, k_max, False)
    f32, G = cfg.dtype == "f32", cfg.Hq // cfg.Hkv
    assert rules(f"order {G} {k_max} {P} 0 0", f"first {f32:d} {G} {W} {k_max} 0") == [order, first]
    rng = np.random.default_rng(k_max)
    idx, cnt = np.full((B, cfg.Hq, k_max), -1, np.int32), np.zeros((B, cfg.Hq), np.int32)
    for b in range(B):
        shared = rng.permutation(P)[:k_max // 2]                 # the heads of a sequence list these and others
        for h in range(cfg.Hq):
            n = (k_max, k_max - 1, 1, 0)[(b + h) % 4]
            some = np.unique(np.concatenate([shared, rng.choice(P, k_max, replace=False)]))
            idx[b, h, :n] = np.sort(rng.permutation(some)[:n])
            cnt[b, h] = n
    D = runner.DeviceLayer.upload(L)
    step = runner.HybridStep(D.shape, W, P, k_max)
    step.idx.copy_(torch.from_numpy(idx))
    step.cnt.copy_(torch.from_numpy(cnt))
    hgca.hybrid_decode_step_selected(D.shape, D.q, D.window, D.pool, step.idx, step.cnt, k_max, step.o, step.lse, step.ws_dense,
                                     step.ws_sparse)
    torch.cuda.synchronize()
    tier = lambda t: oracle.Tier(t.k, t.v, t.cap, t.seq_lens, t.block_table, t.block_size)
    o, lse = oracle.attend_union(L.q, tier(L.window), tier(L.pool), idx, cnt, L.scale)
    compare(step.o, step.lse, o, lse, 1e-5 if f32 else 2e-4)
