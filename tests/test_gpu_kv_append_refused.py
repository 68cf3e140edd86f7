"""More tokens than any window can take: the sequence receives none, the status bit is raised, and nothing of what was announced
is read -- not even where its number of pieces is beyond 32 bits, as a caller's mistake may make it."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_tokens", [33, 20_000_000, 2**31 - 1])
def test_refused_whole(n_tokens):
    import torch
    from paper_2507_03153_amd import cache, hgca
    C = cache.LayerCache(torch.bfloat16, 2, 4, 2, 128, 16, 2, 4, 16, 0.1)
    g = torch.Generator(device="cuda").manual_seed(3)
    C.k_blocks.normal_(generator=g)
    C.v_blocks.normal_(generator=g)
    C.win_lens.copy_(torch.tensor([0, 17], dtype=torch.int32))
    before = [t.clone() for t in (C.k_blocks, C.v_blocks, C.win_lens, C.pool_lens)]
    rows = torch.randn(2, 33, 2, 128, generator=g, device="cuda").to(torch.bfloat16)
    rc = hgca.lib().hgca_kv_append_tokens(ctypes.byref(C.shape), ctypes.byref(C.state), rows.data_ptr(), rows.data_ptr(), n_tokens,
                                          None, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == 0 and int(C.status.cpu()[0]) == hgca.CACHE_WINDOW_FULL
    assert all(torch.equal(a, b) for a, b in zip((C.k_blocks, C.v_blocks, C.win_lens, C.pool_lens), before))
