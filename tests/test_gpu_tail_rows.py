"""The tail of a managed decode step: 1024 threads per row up to 256 rows, 256 threads beyond.  Both fold the same partials and
update the same averages, so sequences of a large batch get what they get in a small one, across evictions."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,win_blocks", [("bf16", 128, 5), ("f32", 64, 5), ("bf16", 64, 300)], ids=["bf16", "f32", "long_window"])
def test_rows_of_large_and_small_launches_agree(dtype, d, win_blocks):
    import torch
    from paper_2507_03153_amd import hgca
    from paper_2507_03153_amd.cache import LayerCache
    hgca.lib()
    dev, dt, Hq, Hkv, bs, steps, some = "cuda:0", torch.bfloat16 if dtype == "bf16" else torch.float32, 8, 2, 16, 20, 3
    B = 256 // Hq + 1                                            # one sequence more than the large workgroups take
    g = torch.Generator(device=dev).manual_seed(5)
    n0 = win_blocks * bs - torch.randint(1, 18, (B,), generator=g, device=dev)
    rnd = lambda *s: torch.randn(*s, generator=g, device=dev)
    blocks = rnd(B, win_blocks + 4, 2, Hkv, bs, d).to(dt)
    maw, q, k, v = rnd(B, Hq, win_blocks * bs).abs() / (win_blocks * bs), rnd(steps, B, Hq, d).to(dt), rnd(steps, B, Hkv, d).to(dt), rnd(steps, B, Hkv, d).to(dt)

    def run(n):
        C = LayerCache(dt, n, Hq, Hkv, d, bs, win_blocks, win_blocks + 4, 64, d ** -0.5, dev)
        C.block_table.copy_(torch.arange(C.block_table.numel(), dtype=torch.int32, device=dev).view(n, -1))
        C.k_blocks.view(n, win_blocks + 4, Hkv, bs, d).copy_(blocks[:n, :, 0])
        C.v_blocks.view(n, win_blocks + 4, Hkv, bs, d).copy_(blocks[:n, :, 1])
        C.win_lens.copy_(n0[:n])
        C.a_maw.zero_()
        C.a_maw[:, :, : maw.shape[2]].copy_(maw[:n])
        out = []
        for t in range(steps):
            C.decode_step(q[t, :n].contiguous(), k[t, :n].contiguous(), v[t, :n].contiguous(), 0.3, 1.0, one_call=True)
            out.append([x[:some].clone() for x in (C.o, C.lse, C.a_gpu, C.a_maw, C.ctx_idx, C.ctx_cnt, C.win_lens, C.pool_lens)])
        torch.cuda.synchronize()
        return out, C

    large, CL = run(some)                                        # 24 rows
    small, CS = run(B)                                           # 264 rows
    assert int(CL.pool_lens.max()) > 0, "no eviction happened"
    listed = 0
    for t, (x, y) in enumerate(zip(large, small)):
        for name, a, b in zip(("o", "lse", "a_gpu", "a_maw"), x, y):
            # both launches may cut the window into other splits: fp32 sums in another order
            assert torch.allclose(a, b, rtol=2e-5, atol=2e-6), (t, name, float((a - b).abs().max()))
        for name, a, b in zip(("win_lens", "pool_lens"), x[6:], y[6:]):
            assert torch.equal(a, b), (t, name)
        assert float((x[5] - y[5]).abs().max()) <= 1             # an average that stands at the threshold
        for b in range(some):
            for h in range(Hq):
                p, r = (z[4][b, h, : int(z[5][b, h])] for z in (x, y))
                for z in (p, r):                                 # in order, and of the pool
                    assert bool((z[1:] > z[:-1]).all()) and (z.numel() == 0 or (int(z[0]) >= 0 and int(z[-1]) < int(x[7][b]))), (t, b, h)
                assert len(set(p.tolist()) ^ set(r.tolist())) <= 1, (t, b, h)
                listed += len(p)
    assert listed > 100, "next to nothing was listed"
