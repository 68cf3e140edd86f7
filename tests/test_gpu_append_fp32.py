"""fp32 append stage on the matrix instructions and query by query, against a 64-bit reference that gives every query exactly the tokens
it sees."""
import numpy as np
import pytest

from routes_rules import rules, runs_query_by_query  # noqa: F401
from test_gpu_append import gpu, to_paged  # noqa: F401

pytestmark = pytest.mark.gpu


def reference(q, K, V, lens, scale, causal):
    """O and lse in 64 bits, each query over the rows it sees and no others (a row holding inf or NaN then reaches the
    queries that see it and no others)."""
    B, N, Hq, d = q.shape
    G = Hq // K.shape[1]
    o, lse = np.zeros((B, N, Hq, d)), np.full((B, N, Hq), -np.inf)
    for b in range(B):
        for i in range(N):
            n = max(int(lens[b]) - N + i + 1, 0) if causal else int(lens[b])
            for h in range(Hq):
                if n == 0:
                    continue
                k, v = K[b, h // G, :n].astype(np.float64), V[b, h // G, :n].astype(np.float64)
                s = (k @ q[b, i, h].astype(np.float64)) * scale
                p = np.exp(s - s.max())
                lse[b, i, h] = s.max() + np.log(p.sum())
                with np.errstate(invalid="ignore"):
                    o[b, i, h] = (p[:, None] * v).sum(0) / p.sum()
    return o, lse


@pytest.mark.parametrize("causal", [True, False], ids=["causal", "whole"])
@pytest.mark.parametrize("kw", [
    dict(B=2, N=100, Hq=8, Hkv=2, d=128, cap=203, lens=(203, 133)),          # four blocks of rows, steps cut by the length
    dict(B=2, N=150, Hq=4, Hkv=4, d=64, cap=256, lens=(256, 193)),
    dict(B=1, N=33, Hq=8, Hkv=1, d=128, cap=1024, lens=(1011,), paged=True),
    # few enough rows, or tokens, to run query by query
    dict(B=1, N=33, Hq=8, Hkv=1, d=128, cap=192, lens=(192,), paged=True, by_query=True),
    dict(B=2, N=40, Hq=8, Hkv=2, d=128, cap=203, lens=(203, 70), by_query=True),
    dict(B=2, N=20, Hq=4, Hkv=4, d=64, cap=128, lens=(128, 65), by_query=True),
], ids=["gqa4", "mha_d64", "gqa8_paged", "gqa8_paged_few", "gqa4_few", "mha_d64_few"])
def test_rows_a_query_does_not_see_may_hold_anything(gpu, rules, kw, causal):  # noqa: F811
    """Infinities and NaNs in V rows behind a query's causal limit, and in the last row of a tier whose length is no
    whole number of steps: O of a query is what its own rows give."""
    torch, hgca, runner = gpu
    B, N, Hq, Hkv, d, cap, lens = (kw[x] for x in ("B", "N", "Hq", "Hkv", "d", "cap", "lens"))
    assert runs_query_by_query(rules, B, N, Hq, Hkv, d, cap) == kw.get("by_query", False)
    lens = np.array(lens, np.int32)
    rng = np.random.default_rng(3)
    q, K, V = (rng.standard_normal(s).astype(np.float32) for s in ((B, N, Hq, d), (B, Hkv, cap, d), (B, Hkv, cap, d)))
    for b, n in enumerate(lens):
        V[b, :, n - 1, ::2] = np.inf                             # seen by the last query only, where causal
        V[b, 0, n - 3, 1::4] = np.nan
        V[b, -1, n - N // 2, :5] = -np.inf
        V[b, :, n:] = np.nan                                     # behind the end: nobody's
        K[b, :, n:] = np.nan
    g = lambda a: runner._to_gpu(a, "cuda:0")
    shape = hgca.Shape(hgca.F32, B, Hq, Hkv, d, d ** -0.5)
    tier = to_paged(runner, hgca, torch, K, V, lens, cap, 16, 4, "cuda:0") if kw.get("paged") else \
        hgca.Tier(g(K), g(V), cap, g(lens))
    o, lse = torch.zeros(B, N, Hq, d, device="cuda:0"), torch.zeros(B, N, Hq, device="cuda:0")
    hgca.append_attn(shape, g(q), tier, causal, o, lse, hgca.append_workspace(shape, N, cap, "cuda:0"))
    torch.cuda.synchronize()
    o_ref, l_ref = reference(q, K, V, lens, d ** -0.5, causal)
    o, lse = o.cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64)
    assert np.max(np.abs(lse - l_ref)) <= 1e-5
    finite = np.isfinite(o_ref)
    assert finite.any() and not finite.all()
    assert np.array_equal(np.isfinite(o), finite), f"{np.sum(np.isfinite(o) != finite)} of {o.size} outputs differ in kind"
    assert np.array_equal(np.isnan(o), np.isnan(o_ref)) and np.array_equal(o[np.isinf(o_ref)], o_ref[np.isinf(o_ref)])
    assert np.max(np.abs(o[finite] - o_ref[finite])) <= 1e-5


@pytest.mark.parametrize("kw", [
    # few queries, one by one
    dict(B=1, N=1, Hq=8, Hkv=8, d=128, cap=700, lens=(700,), by_query=True),
    dict(B=2, N=3, Hq=8, Hkv=2, d=128, cap=300, lens=(300, 2), by_query=True),
    dict(B=3, N=16, Hq=4, Hkv=4, d=64, cap=256, lens=(256, 16, 3), by_query=True),
    dict(B=2, N=2, Hq=16, Hkv=4, d=128, cap=2048, lens=(2048, 1500), by_query=True),
    dict(B=2, N=3, Hq=16, Hkv=4, d=64, cap=1008, lens=(1000, 1), paged=True, by_query=True),
    dict(B=1, N=20, Hq=16, Hkv=2, d=128, cap=160, lens=(150,), paged=True, by_query=True),
    # on the matrix instructions
    dict(B=2, N=5, Hq=8, Hkv=1, d=64, cap=130, lens=(130, 77), paged=True),
    dict(B=2, N=2, Hq=16, Hkv=2, d=128, cap=1000, lens=(1000, 0)), dict(B=2, N=48, Hq=16, Hkv=2, d=128, cap=1000, lens=(1000, 513)),
    dict(B=1, N=70, Hq=8, Hkv=4, d=128, cap=3000, lens=(2999,)),             # 140 rows
], ids=["n1", "n3_short", "n16_d64", "n2_gqa4", "n3_gqa4_paged", "n20_gqa8_paged", "n5_paged", "n2_empty", "n48_gqa8", "n70"])
@pytest.mark.parametrize("causal", [True, False], ids=["causal", "whole"])
def test_either_route(gpu, rules, kw, causal):  # noqa: F811
    torch, hgca, runner = gpu
    B, N, Hq, Hkv, d, cap, lens = (kw[x] for x in ("B", "N", "Hq", "Hkv", "d", "cap", "lens"))
    assert runs_query_by_query(rules, B, N, Hq, Hkv, d, cap) == kw.get("by_query", False)
    lens = np.array(lens, np.int32)
    rng = np.random.default_rng(N)
    q, K, V = (rng.standard_normal(s).astype(np.float32) for s in ((B, N, Hq, d), (B, Hkv, cap, d), (B, Hkv, cap, d)))
    g = lambda a: runner._to_gpu(a, "cuda:0")
    shape = hgca.Shape(hgca.F32, B, Hq, Hkv, d, d ** -0.5)
    tier = to_paged(runner, hgca, torch, K, V, lens, cap, 16, 4, "cuda:0") if kw.get("paged") else \
        hgca.Tier(g(K), g(V), cap, g(lens))
    o, lse = torch.full((B, N, Hq, d), float("nan"), device="cuda:0"), torch.full((B, N, Hq), float("nan"), device="cuda:0")
    hgca.append_attn(shape, g(q), tier, causal, o, lse, hgca.append_workspace(shape, N, cap, "cuda:0"))
    torch.cuda.synchronize()
    o_ref, l_ref = reference(q, K, V, lens, d ** -0.5, causal)
    o, lse = o.cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64)
    empty = np.isneginf(l_ref)
    assert np.array_equal(np.isneginf(lse), empty) and np.all(o[empty] == 0)
    assert np.max(np.abs(lse[~empty] - l_ref[~empty])) <= 1e-5 and np.max(np.abs(o - o_ref)) <= 1e-5


def test_few_queries_over_more_splits_than_the_workspace_holds(gpu):  # noqa: F811
    """One query over 4096 tokens and 16 (sequence, KV head) pairs would be cut into more splits than the workspace of the
    call has slots: its splits are longer then."""
    torch, hgca, runner = gpu
    B, N, Hq, Hkv, d, cap = 2, 1, 32, 8, 128, 4096
    g = torch.Generator(device="cuda:0").manual_seed(2)
    q, k, v = (torch.randn(*s, generator=g, device="cuda:0") for s in ((B, N, Hq, d), (B, Hkv, cap, d), (B, Hkv, cap, d)))
    o, lse = torch.zeros(B, N, Hq, d, device="cuda:0"), torch.zeros(B, N, Hq, device="cuda:0")
    shape = hgca.Shape(hgca.F32, B, Hq, Hkv, d, d ** -0.5)
    hgca.append_attn(shape, q, hgca.Tier(k, v, cap), False, o, lse, hgca.append_workspace(shape, N, cap, "cuda:0"))
    torch.cuda.synchronize()
    o_ref, l_ref = reference(q.cpu().numpy(), k.cpu().numpy(), v.cpu().numpy(), [cap] * B, d ** -0.5, False)
    assert np.max(np.abs(o.cpu().numpy() - o_ref)) <= 1e-5 and np.max(np.abs(lse.cpu().numpy() - l_ref)) <= 1e-5


@pytest.mark.parametrize("kw", [
    dict(B=2, Hq=8, Hkv=2, d=128, seed=41), dict(B=1, Hq=16, Hkv=2, d=128, seed=42), dict(B=2, Hq=4, Hkv=4, d=64, seed=43),
], ids=["gqa4", "gqa8", "mha_d64"])
def test_turns_over_a_long_line(kw):
    """Managed turns: pool and window as one line of tokens in fp32, an empty pool at first and some thousand tokens at last,
    up to 8000 query rows per KV head (the weights pass adds to its output block after block of them)."""
    import torch
    from paper_2507_03153_amd import cache, hgca, runner
    from test_gpu_kv_turns import run_turns
    hgca.lib()
    prefill = (0, 100)[:kw["B"]]
    _, _, status, st = run_turns((torch, hgca, runner, cache), block_size=16, win_blocks=8, max_blocks=200, k_max=2900,
                                 turns=[("a", 1000), ("a", 900), ("d", 3), ("a", 700), ("a", 40), ("a", 33)], alpha=0.3, beta=1.0,
                                 prefill=prefill, fp32=True, **kw)
    assert status == 0 and st["evicted_blocks"] >= 40
