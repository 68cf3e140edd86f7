"""Decode steps short enough for the two-launch path of hgca_hybrid_decode_step (window splits with the score pass;
selection, attention over the list and fold per row), at the edges of its rule and of its loops: lists of 0, 1, a whole
load round and one more, every entry; empty and one-token windows and pools; window partials in one, a whole and more than
one pass of the fold.  The selection has to equal the separate call's, outputs the oracle's.  Bars as in test_gpu_parity:
fp32 accumulation over exact products."""
import numpy as np
import pytest

from paper_2507_03153_amd import workloads as wl

pytestmark = pytest.mark.gpu

# up to 256 rows and budgets of up to 128 KB (bf16) or 384 KB (fp32) of V rows take the short path; "over" cases lie behind the edge of
# the budget (the edges of the rows and of the keys are in test_gpu_step_routes)
CASES = [
    ("bf16_gqa4", "C2", dict(Hq=8, Hkv=2), 1024, 3000, 512),
    ("bf16_gqa4_over", "C2", dict(Hq=8, Hkv=2), 1024, 3000, 513),
    ("bf16_mha_d64", "C2", dict(Hq=4, Hkv=4, d=64), 200, 2500, 1024),
    ("bf16_gqa8", "C2", dict(Hq=16, Hkv=2), 4500, 1000, 257),
    ("bf16_gqa2_paged", "C5", dict(Hq=4, Hkv=2), 300, 1700, 130),
    ("bf16_long_rows", "C2", dict(Hq=4, Hkv=4, d=64), 100, 36000, 300),
    ("f32_gqa4", "C1", dict(Hq=8, Hkv=2), 700, 2000, 129),
    ("f32_d128_over", "C1", dict(Hq=2, Hkv=1, d=128), 2300, 1500, 769),
    ("f32_d128", "C1", dict(Hq=2, Hkv=1, d=128), 2300, 1500, 768),
    ("f32_gqa8_paged", "C1", dict(Hq=8, Hkv=1, block_size=16), 90, 400, 65),
]


@pytest.mark.parametrize("name,kw,W,P,k_max", [c[1:] for c in CASES], ids=[c[0] for c in CASES])
def test_short_step_equals_the_oracle(oracle, name, kw, W, P, k_max):
    import torch
    from paper_2507_03153_amd import hgca, runner
    ks = [k_max, k_max - 1, 1, 0, k_max, 64, k_max]
    w_lens = [W, 1, 64, W - 1, 0, 65, W]
    p_lens = [P, P - 1, 1, 77, min(k_max, P), 63, 0]
    cfg = wl.scaled(wl.CONFIGS[name], B=len(ks), W=W, P=P, k=16, ragged=None, **kw)
    L = wl.make_layer(cfg)
    L.window.seq_lens, L.pool.seq_lens = np.array(w_lens, np.int32), np.array(p_lens, np.int32)
    D = runner.DeviceLayer.upload(L)
    step = runner.HybridStep(D.shape, cfg.W, cfg.P, k_max)
    k_dev = torch.tensor(ks, dtype=torch.int32, device="cuda")
    tier = lambda t: oracle.Tier(t.k, t.v, t.cap, t.seq_lens, t.block_table, t.block_size)
    o, lse, idx, cnt = oracle.hybrid_step(L.q, tier(L.window), tier(L.pool), np.array(ks, np.int32), k_max, L.scale)
    sel_idx, sel_cnt = torch.empty_like(step.idx), torch.empty_like(step.cnt)
    hgca.select_salient(D.shape, D.q, D.pool, k_dev, k_max, sel_idx, sel_cnt, step.ws_sparse)
    tol = 1e-5 if cfg.dtype == "f32" else 2e-4
    for o_dtype in (torch.float32, torch.bfloat16):
        out = torch.empty(step.o.shape, dtype=o_dtype, device="cuda")
        for _ in range(2):                       # the second call meets the first one's workspace
            hgca.hybrid_decode_step(D.shape, D.q, D.window, D.pool, k_dev, k_max, step.idx, step.cnt, out, step.lse,
                                    step.ws_dense, step.ws_sparse)
        torch.cuda.synchronize()
        assert torch.equal(step.idx, sel_idx) and torch.equal(step.cnt, sel_cnt)
        assert np.array_equal(step.cnt.cpu().numpy(), cnt)
        got_l = step.lse.double().cpu().numpy()
        assert np.array_equal(np.isinf(got_l), np.isinf(lse))
        some = np.isfinite(lse)
        assert np.max(np.abs(got_l[some] - lse[some])) <= tol
        bar = tol if o_dtype == torch.float32 else tol + np.max(np.abs(o)) * 2.0 ** -8   # one rounding to bf16
        assert np.max(np.abs(out.double().cpu().numpy() - o)) <= bar


@pytest.mark.parametrize("name,kw,W,P,k_max", [
    ("C2", dict(Hq=8, Hkv=2), 300, 900, 200), ("C5", dict(Hq=4, Hkv=2), 100, 1700, 130), ("C1", dict(Hq=8, Hkv=2), 90, 2000, 129),
    ("C2", dict(Hq=4, Hkv=4, d=64), 100, 36000, 300),
], ids=["bf16", "bf16_paged", "f32", "bf16_long_rows"])
def test_queries_that_are_not_numbers(name, kw, W, P, k_max):
    """One head's query is NaN, and so is every score of its row: the positions in its list and the rows that are read stay
    inside the sequence whatever the list held before, and the other heads' results are those without it, bit for bit."""
    import torch
    from paper_2507_03153_amd import hgca, runner
    p_lens = [P, 65, k_max, 1, 0]                # with 1 and k_max valid positions every one is kept
    cfg = wl.scaled(wl.CONFIGS[name], B=len(p_lens), W=W, P=P, k=16, ragged=None, **kw)
    L = wl.make_layer(cfg)
    L.pool.seq_lens = np.array(p_lens, np.int32)
    D = runner.DeviceLayer.upload(L)
    step = runner.HybridStep(D.shape, cfg.W, cfg.P, k_max)
    bad = 1
    outs = []
    for q, left in ((D.q, -1), (D.q.clone(), -1), (D.q.clone(), 0x7fffff00), (D.q.clone(), -0x7fffff00)):
        if outs:
            q[:, bad] = float("nan")
        step.idx.fill_(left)
        hgca.hybrid_decode_step(D.shape, q, D.window, D.pool, min(k_max, P), k_max, step.idx, step.cnt, step.o, step.lse,
                                step.ws_dense, step.ws_sparse)
        torch.cuda.synchronize()
        outs.append([t.clone() for t in (step.idx, step.cnt, step.o, step.lse)])
    good = [h for h in range(cfg.Hq) if h != bad]
    for got in outs[1:]:
        for x, want in zip(got, outs[0]):
            assert torch.equal(x[:, good], want[:, good])
        assert torch.equal(got[1], outs[0][1])
