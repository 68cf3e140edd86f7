"""A turn over a managed cache of 512 MB and more leaves part of K to the caches between attention and weights, and the weights pass
walks the passes of its shares from the end: same values as the two calls by themselves, bit for bit, whatever the lengths."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,G,blocks,n_q,lens", [
    (64, 4, 16336, 32, [(5000, 200), (0, 33)]),          # 512 MB, 12 sixteenths; an empty pool; steps and tiles that lengths cut
    (128, 2, 16336, 5, [(16, 64), (70000, 500)]),        # 1 GB, 8 sixteenths; a share of one tile; several waves to a tile
    (64, 8, 16335, 16, [(4096, 128), (31, 47)]),         # one block less: everything streamed, from the start
], ids=["d64", "d128", "below"])
def test_turn_is_its_parts(d, G, blocks, n_q, lens):
    import torch
    from paper_2507_03153_amd import hgca
    from paper_2507_03153_amd.cache import LayerCache
    hgca.lib()
    dev, dt, B, Hkv, bs, win_blocks = "cuda:0", torch.bfloat16, 2, 4, 16, 48
    Hq = Hkv * G
    g = torch.Generator(device=dev).manual_seed(11)
    C = LayerCache(dt, B, Hq, Hkv, d, bs, win_blocks, blocks, 64, d ** -0.5, dev)
    assert ((C.win_cap + C.pool_cap) * B * Hkv * d * 4 >= 512 << 20) == (blocks == 16336)
    C.k_blocks.normal_(generator=g)
    C.v_blocks.normal_(generator=g)
    q = torch.randn(B, n_q, Hq, d, generator=g, device=dev).to(dt)
    k_in, v_in = (torch.randn(B, n_q, Hkv, d, generator=g, device=dev).to(dt) for _ in range(2))
    pool = torch.tensor([p // bs * bs for p, _ in lens], dtype=torch.int32, device=dev)
    win = torch.tensor([w for _, w in lens], dtype=torch.int32, device=dev)

    def place():
        C.block_table.copy_(torch.arange(B * blocks, dtype=torch.int32, device=dev).view(B, blocks).flip(1))
        C.pool_lens.copy_(pool)
        C.win_lens.copy_(win)
        C.first_win_block.copy_(pool // bs)
        C.a_maw.zero_()
        C.append_buffers(n_q)
        for x in (C.a_gpu, C.a_cpu, C.o_app, C.lse_app):
            x.fill_(7.0)

    place()
    hgca.kv_append_tokens(C.shape, C.state, k_in, v_in)
    ws = hgca.append_tiers_workspace(C.shape, n_q, C.win_cap, C.pool_cap, dev)
    lse_w, lse_p = torch.empty_like(C.lse_app), torch.empty_like(C.lse_app)
    hgca.append_attn_tiers(C.shape, q, C.window, C.pool, C.o_app, C.lse_app, ws, lse_w, lse_p)
    hgca.append_weights_tiers(C.shape, q, C.window, C.pool, lse_w, lse_p, C.a_gpu, C.a_cpu)
    parts = [x.clone() for x in (C.o_app, C.lse_app, C.a_gpu, C.a_cpu)]
    place()
    C.append_step(q, k_in, v_in, 0.3, 4.0)
    torch.cuda.synchronize()
    for name, x, y in zip(("o", "lse", "a_gpu", "a_cpu"), (C.o_app, C.lse_app, C.a_gpu, C.a_cpu), parts):
        assert torch.equal(x, y), (name, float((x - y).abs().max()))
    for b in range(B):                                   # a query that sees all weighs to 1 over both tiers
        assert abs(float(C.a_gpu[b].sum(1).mean()) - 1) < 1e-3 and (pool[b] == 0 or abs(float(C.a_cpu[b].sum(1).mean()) - 1) < 1e-3)
