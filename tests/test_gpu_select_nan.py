"""Selection on rows that hold NaN, which ranks as -inf: the list is the one of the row with -inf in its place, whole and
valid, whatever the list held before; the kept scores are the row's own."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# the lengths at which the selection changes its way of holding a row, in large and in small workgroups
@pytest.mark.parametrize("n_rows,cap", [(6, 700), (6, 16381), (6, 33795), (6, 61003), (6, 135168), (6, 135171),
                                        (300, 700), (300, 4099), (300, 14337), (300, 30000)])
def test_rows_with_nan(oracle, n_rows, cap):
    import torch
    from paper_2507_03153_amd import hgca
    rng = np.random.default_rng(cap + n_rows)
    scores = rng.standard_normal((1, n_rows, cap)).astype(np.float32)
    some = rng.permutation(cap)
    scores[0, 0] = np.nan                                        # nothing but NaN
    scores[0, 1, some[:20]] = np.nan                             # a few: fewer numbers than wanted, if nearly all are
    scores[0, 2, rng.random(cap) < 0.3] = np.nan
    scores[0, 3, some[:30]], scores[0, 3, some[30:60]] = np.nan, -np.inf     # ties of the two, by position
    scores[0, 4] = -np.abs(scores[0, 4])                         # no score above zero
    scores[0, 4, some[:20]] = np.nan
    shape = hgca.Shape(hgca.F32, 1, n_rows, n_rows, 128, 1.0)
    d = torch.from_numpy(scores).cuda()
    for k in (1, cap // 20, cap // 2, cap - 25, cap - 10, cap - 1):
        idx = torch.full((1, n_rows, k), 0x7fffff00, dtype=torch.int32, device="cuda")
        cnt, sel = torch.zeros(1, n_rows, dtype=torch.int32, device="cuda"), torch.zeros(1, n_rows, k, device="cuda")
        hgca.select_topk(shape, d, None, cap, k, k, idx, cnt, sel_scores_out=sel)
        torch.cuda.synchronize()
        want, want_cnt = oracle.select_given(np.where(np.isnan(scores), np.float32(-np.inf), scores), k, k)
        assert np.array_equal(cnt.cpu().numpy(), want_cnt)
        for r in range(n_rows):
            assert np.array_equal(idx.cpu().numpy()[0, r], want[0, r]), (k, r)
        assert np.array_equal(sel.cpu().numpy(), np.take_along_axis(scores, want.astype(np.int64), axis=2), equal_nan=True)
