"""fp32 append stage with products of bf16 parts: edges of its tiles (16 rows, 32 tokens), values that have no parts, and
its error against 64 bits."""
import numpy as np
import pytest

from routes_rules import rules, runs_query_by_query  # noqa: F401
from test_gpu_append import gpu, to_paged  # noqa: F401
from test_gpu_append_fp32 import reference

pytestmark = pytest.mark.gpu


def weights_reference(q, K, lens, lse, scale, causal, cap):
    B, N, Hq, d = q.shape
    G = Hq // K.shape[1]
    a = np.zeros((B, Hq, cap))
    for b in range(B):
        for i in range(N):
            n = max(int(lens[b]) - N + i + 1, 0) if causal else int(lens[b])
            for h in range(Hq):
                a[b, h, :n] += np.exp((K[b, h // G, :n].astype(np.float64) @ q[b, i, h].astype(np.float64)) * scale - lse[b, i, h])
    return a / N


def run(gpu, rules, q, K, V, lens, causal, paged, scale=None):  # noqa: F811
    torch, hgca, runner = gpu
    B, N, Hq, d = q.shape
    Hkv, cap = K.shape[1:3]
    assert not runs_query_by_query(rules, B, N, Hq, Hkv, d, cap), "a capacity at which the call takes the matrix instructions"
    g = lambda a: runner._to_gpu(a, "cuda:0")
    shape = hgca.Shape(hgca.F32, B, Hq, Hkv, d, d ** -0.5 if scale is None else scale)
    tier = to_paged(runner, hgca, torch, K, V, lens, cap, 16, 4, "cuda:0") if paged else hgca.Tier(g(K), g(V), cap, g(lens))
    o, lse = torch.full((B, N, Hq, d), float("nan"), device="cuda:0"), torch.full((B, N, Hq), float("nan"), device="cuda:0")
    a = torch.full((B, Hq, cap), float("nan"), device="cuda:0")
    hgca.append_attn(shape, g(q), tier, causal, o, lse, hgca.append_workspace(shape, N, cap, "cuda:0"))
    hgca.append_weights(shape, g(q), tier, causal, lse, a)
    torch.cuda.synchronize()
    return (x.cpu().numpy().astype(np.float64) for x in (o, lse, a))


@pytest.mark.parametrize("causal", [True, False], ids=["causal", "whole"])
@pytest.mark.parametrize("kw", [
    dict(N=60, Hq=4, Hkv=4, d=64, lens=(31, 33)), dict(N=64, Hq=4, Hkv=2, d=128, lens=(32, 65)),         # 60 and 128 rows
    dict(N=31, Hq=8, Hkv=2, d=128, lens=(64, 1), paged=True), dict(N=17, Hq=16, Hkv=2, d=128, lens=(97, 129)),   # 124, 136
    dict(N=16, Hq=16, Hkv=2, d=64, lens=(700, 481)), dict(N=65, Hq=8, Hkv=4, d=64, lens=(300, 95), paged=True),  # 128, 130
], ids=["mha_d64", "gqa2", "gqa4_paged", "gqa8", "gqa8_d64", "gqa2_d64_paged"])
def test_edges_of_tiles(gpu, rules, kw, causal):  # noqa: F811
    N, Hq, Hkv, d, lens = (kw[x] for x in ("N", "Hq", "Hkv", "d", "lens"))
    lens, cap, B = np.array(lens, np.int32), max(kw["lens"]) + 905, 2
    rng = np.random.default_rng(N)
    q, K, V = (rng.standard_normal(s).astype(np.float32) for s in ((B, N, Hq, d), (B, Hkv, cap, d), (B, Hkv, cap, d)))
    o, lse, a = run(gpu, rules, q, K, V, lens, causal, kw.get("paged"))
    o_ref, l_ref = reference(q, K, V, lens, d ** -0.5, causal)
    empty = np.isneginf(l_ref)
    assert np.array_equal(np.isneginf(lse), empty) and np.all(o[empty] == 0)
    assert np.max(np.abs(lse[~empty] - l_ref[~empty])) <= 1e-5 and np.max(np.abs(o - o_ref)) <= 1e-5
    a_ref = weights_reference(q, K, lens, np.where(empty, 0.0, l_ref), d ** -0.5, causal, cap)
    assert np.max(np.abs(a - a_ref)) <= 1e-5


@pytest.mark.parametrize("kw", [dict(N=40, Hq=8, Hkv=2, d=128), dict(N=40, Hq=16, Hkv=2, d=64), dict(N=130, Hq=4, Hkv=4, d=64)],
                         ids=["gqa4", "gqa8_d64", "mha_d64"])
def test_values_without_parts(gpu, rules, kw):  # noqa: F811
    """Keys with an infinite component that every query meets with the same sign (their scores are -inf: they weigh nothing),
    keys whose products overflow a part but not the sum's type, and V entries that round to infinity in 16 bits."""
    N, Hq, Hkv, d = (kw[x] for x in ("N", "Hq", "Hkv", "d"))
    B, cap, lens = 2, 760, np.array((260, 201), np.int32)
    rng = np.random.default_rng(d)
    q, K, V = (rng.standard_normal(s).astype(np.float32) for s in ((B, N, Hq, d), (B, Hkv, cap, d), (B, Hkv, cap, d)))
    q[..., 0], q[..., 1] = 1.0, 1e-38
    K[..., 0] = 0.0
    K[:, :, 3::17, 0] = -np.inf
    K[:, :, 5::19, 1] = np.float32(3.4e38)                       # times 1e-38: 3.4, an ordinary term of the score
    # finite, but its upper part is not.  One to a column: a weight is at most 1 before the sum is divided, so one such entry
    # stays below the largest fp32 number (3.4028e38), and the sum of several may not, whatever forms their products.
    for i in range(8):
        V[:, :, 2 + 23 * i, 3 + i] = np.float32(3.4e38)
    o, lse, a = run(gpu, rules, q, K, V, lens, False, False)
    o_ref, l_ref = reference(q, K, V, lens, d ** -0.5, False)
    assert np.max(np.abs(lse - l_ref)) <= 1e-5
    assert np.max(np.abs(o - o_ref) / np.maximum(np.abs(o_ref).max(axis=(0, 1, 2)), 1.0)) <= 1e-5
    a_ref = weights_reference(q, K, lens, l_ref, d ** -0.5, False, cap)
    assert np.max(np.abs(a - a_ref)) <= 1e-5 and np.all(a[:, :, 3:200:17] == 0)


@pytest.mark.parametrize("case", ["large_and_small", "small_queries", "small_keys", "small_scale", "small_values", "small_weights", "low_scores"])
@pytest.mark.parametrize("kw", [dict(N=40, Hq=8, Hkv=2, d=128), dict(N=100, Hq=4, Hkv=4, d=64)], ids=["gqa4", "mha_d64"])
def test_ends_of_the_range(gpu, rules, kw, case):  # noqa: F811
    """Normal fp32 operands whose lower parts bf16 has no bits for: what they give is as exact as anywhere else."""
    N, Hq, Hkv, d = (kw[x] for x in ("N", "Hq", "Hkv", "d"))
    B, cap, lens, scale = 2, 760, np.array((260, 201), np.int32), d ** -0.5
    rng = np.random.default_rng(d)
    q, K, V = (rng.standard_normal(s) for s in ((B, N, Hq, d), (B, Hkv, cap, d), (B, Hkv, cap, d)))
    if case == "large_and_small":                                # 3e38 has a bf16 part of its own; the terms are up to 3
        q[..., 1] *= 1e-38
        K[..., 1] = 0.0
        K[:, :, 5::19, 1] = 3e38
    elif case in ("small_queries", "small_keys", "small_scale"):
        a, b = {"small_queries": (-119, 14), "small_keys": (14, -119), "small_scale": (60, 41)}[case]
        q, K, scale = q * 2.0 ** a, K * 2.0 ** b, scale * 2.0 ** -(a + b)
    elif case == "small_values":
        V[..., ::3] *= 2.0 ** -120
    elif case == "small_weights":                                # weights of some 2^-116, all that a column of V has
        K[:, :, 7::11] = 0.0
        q[..., 0], K[..., 0] = d ** 0.5, 82.0
        K[:, :, 7::11, 0] = 0.0
        V[..., 4] = 0.0
        V[:, :, 7::11, 4] = 1e30
    else:                                                        # all scores alike; their products times 2^24 overflow to -inf
        q[...], K[...] = 0.0, 0.0
        q[..., 0], K[..., 0] = 2.0 ** 60, -2.0 ** 50
    q, K, V = (x.astype(np.float32) for x in (q, K, V))
    o, lse, a = run(gpu, rules, q, K, V, lens, False, False, scale)
    scale = float(np.float32(scale))
    o_ref, l_ref = reference(q, K, V, lens, scale, False)
    assert np.max(np.abs(lse - l_ref) / np.maximum(np.abs(l_ref), 1.0)) <= 1e-5
    # a weight that counts lies 80 below the others here: its score is rounded to 80 * 2^-24, and so is the weight
    column = np.abs(o_ref).max(axis=(0, 1, 2))
    assert column.min() > 0 and np.max(np.abs(o - o_ref) / column) <= (4e-5 if case == "small_weights" else 1e-5)
    if case != "low_scores":                                     # (the weights take the rounding of lse, 2^107 here)
        assert np.max(np.abs(a - weights_reference(q, K, lens, l_ref, scale, False, cap))) <= 1e-5


def test_error_against_64_bits(gpu, rules):  # noqa: F811
    """The products of parts are as good as fp32 ones: a score of 128 products is off by a few units of 2^-24 of its terms, and so
    are the weights and O, whose error is that of their scores: 24 queries over 3000 tokens stay below 8 * 2^-24 relative (2-norm)."""
    B, N, Hq, Hkv, d, cap = 1, 24, 4, 2, 128, 3000
    lens = np.array((cap,), np.int32)
    rng = np.random.default_rng(11)
    q, K, V = (rng.standard_normal(s).astype(np.float32) for s in ((B, N, Hq, d), (B, Hkv, cap, d), (B, Hkv, cap, d)))
    q *= 2.0
    o, lse, a = run(gpu, rules, q, K, V, lens, False, False)
    o_ref, l_ref = reference(q, K, V, lens, d ** -0.5, False)
    a_ref = weights_reference(q, K, lens, l_ref, d ** -0.5, False, cap)
    off = lambda x, y: float(np.linalg.norm(x - y) / np.linalg.norm(y))
    print(off(o, o_ref), off(lse, l_ref), off(a, a_ref))
    assert off(o, o_ref) <= 8 * 2.0 ** -24 and off(lse, l_ref) <= 2 * 2.0 ** -24 and off(a, a_ref) <= 8 * 2.0 ** -24


@pytest.mark.parametrize("what", ["v", "k"])
def test_cost_of_values_without_parts(gpu, what):  # noqa: F811
    """What one infinite V entry or one NaN key costs, seen by every query: its shares are worked out again with fp32 products.
    Measured 1.9 and 2.8 times the time without (token by token on the vector units 20 and 29 times); 8 leaves room for noise."""
    torch, hgca, runner = gpu
    B, N, Hq, Hkv, d, cap = 2, 24, 32, 8, 128, 5120
    g = torch.Generator(device="cuda:0").manual_seed(2)
    q, k, v = (torch.randn(*s, generator=g, device="cuda:0") for s in ((B, N, Hq, d), (B, Hkv, cap, d), (B, Hkv, cap, d)))
    shape = hgca.Shape(hgca.F32, B, Hq, Hkv, d, d ** -0.5)
    o, lse, a = (torch.zeros(*s, device="cuda:0") for s in ((B, N, Hq, d), (B, N, Hq), (B, Hq, cap)))

    def best(k, v):
        tier, ws = hgca.Tier(k, v, cap), hgca.append_workspace(shape, N, cap, "cuda:0")
        times = []
        for _ in range(6):
            t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            t[0].record()
            for _ in range(4):
                hgca.append_attn(shape, q, tier, True, o, lse, ws)
                hgca.append_weights(shape, q, tier, True, lse, a)
            t[1].record()
            torch.cuda.synchronize()
            times.append(t[0].elapsed_time(t[1]))
        return min(times)

    without = best(k, v)
    (v if what == "v" else k)[:, :, 7, 3] = float("inf" if what == "v" else "nan")
    again = best(k, v)
    print(what, again / without)
    assert torch.isinf(o[..., 3]).all() if what == "v" else torch.isnan(o).all()
    assert again <= 8 * without


@pytest.mark.parametrize("G,d", [(4, 128), (1, 64)], ids=["gqa4", "mha_d64"])
def test_turn_over_values_without_parts(gpu, G, d):  # noqa: F811
    """A managed turn, both tiers in one launch: an infinite V entry of the pool reaches every query, one of the incoming tokens
    those from its own on, and a key with scores of -inf nobody; weights and the other outputs stay what they are."""
    torch, hgca, runner = gpu
    from paper_2507_03153_amd.cache import LayerCache
    dev, B, Hkv, bs, win_blocks, N = "cuda:0", 2, 2, 16, 12, 20
    Hq, pool, win = Hkv * G, (336, 0), (100, 64)
    g = torch.Generator(device=dev).manual_seed(11)
    C = LayerCache(torch.float32, B, Hq, Hkv, d, bs, win_blocks, win_blocks + 22, 64, d ** -0.5, dev)
    C.block_table.copy_(torch.randperm(C.block_table.numel(), generator=g, device=dev).int().view(B, -1))
    C.k_blocks.normal_(generator=g)
    C.v_blocks.normal_(generator=g)
    C.pool_lens.copy_(torch.tensor(pool))
    C.win_lens.copy_(torch.tensor(win))
    C.first_win_block.copy_(C.pool_lens // bs)
    q = torch.randn(B, N, Hq, d, generator=g, device=dev)
    k_in, v_in = (torch.randn(B, N, Hkv, d, generator=g, device=dev) for _ in range(2))
    q[..., 0] = 1.0
    C.k_blocks[int(C.block_table[0, 5]), :, 7, 0] = -float("inf")
    C.v_blocks[int(C.block_table[0, 9]), :, 3, 5] = float("inf")
    v_in[:, 12, :, 6] = -float("inf")
    rows = lambda x, b, n: x[C.block_table[b].long()].transpose(0, 1).reshape(Hkv, -1, d)[:, :n].double().cpu().numpy()
    old = [[rows(x, b, pool[b] + win[b]) for x in (C.k_blocks, C.v_blocks)] for b in range(B)]
    C.append_buffers(N)
    C.append_step(q, k_in, v_in, 0.3, 4.0)
    torch.cuda.synchronize()
    o, lse, a_cpu, a_gpu = (x.double().cpu().numpy() for x in (C.o_app, C.lse_app, C.a_cpu, C.a_gpu))
    for b in range(B):
        K, V = (np.concatenate((x, y[b].transpose(0, 1).double().cpu().numpy()), 1) for x, y in zip(old[b], (k_in, v_in)))
        n = K.shape[1]
        a_ref = np.zeros((Hq, n))
        o_ref, l_ref = reference(q[b:b + 1].cpu().numpy(), K[None], V[None], [n], d ** -0.5, True)
        for h in range(Hq):
            for i in range(N):                                   # weights of a tier are normalised over the tier
                s = K[h // G] @ q[b, i, h].double().cpu().numpy() * d ** -0.5
                s[n - N + i + 1:] = -np.inf
                for t in (slice(0, pool[b]), slice(pool[b], n)):
                    if t.stop > t.start:
                        p = np.exp(s[t] - s[t].max())
                        a_ref[h, t] += p / p.sum() / N
        finite = np.isfinite(o_ref[0])
        assert np.array_equal(np.isnan(o[b]), np.isnan(o_ref[0])) and np.array_equal(o[b][~finite], o_ref[0][~finite])
        assert (pool[b] == 0 or np.isposinf(o[b, :, :, 5]).all()) and np.isneginf(o[b, 12:, :, 6]).all() and finite[:12, :, 6].all()
        assert np.max(np.abs(o[b][finite] - o_ref[0][finite])) <= 1e-5 and np.max(np.abs(lse[b] - l_ref[0])) <= 1e-5
        assert np.max(np.abs(a_cpu[b, :, :pool[b]] - a_ref[:, :pool[b]]), initial=0) <= 1e-5
        assert np.max(np.abs(a_gpu[b, :, :win[b] + N] - a_ref[:, pool[b]:])) <= 1e-5
