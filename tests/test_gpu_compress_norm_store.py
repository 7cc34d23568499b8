"""Anchor rows of K stored by the similarity GEMM's norm pass: whole rows at their places, nothing behind them, the scores that the chunks
give one at a time (whose anchors are copied beside the selection), and the selection that belongs to them."""
import pytest
import torch

import paper_2605_22718_amd as wk
from wkt import dev

pytestmark = pytest.mark.gpu


# calls on both sides of 20,000,000 bytes of anchor rows; last tokens that leave waves of the norm pass without one
@pytest.mark.parametrize("head_mode", [wk.WK_HEADS_SHARED, wk.WK_HEADS_INDEPENDENT])
@pytest.mark.parametrize("B,H,T,F", [(5, 16, 977, 2), (5, 16, 976, 2), (3, 5, 5209, 3), (80, 1, 979, 2), (9, 9, 965, 1)])
def test_rows_scores_and_selections(B, H, T, F, head_mode):
    d = dev()
    g = torch.Generator(device=d).manual_seed(T)
    K, V = (torch.randn((B, H, F * T, 128), generator=g, device=d).to(torch.bfloat16) for _ in range(2))
    n_out, _ = wk.wk_keep_count(0.25, wk.WK_RATIO_NONANCHOR, wk.WK_ANCHOR_FIRST_FRAME, F, T)
    G = H if head_mode == wk.WK_HEADS_INDEPENDENT else 1

    def call(K, V, guard):
        b = K.shape[0]
        desc = wk.make_compress_desc(H, T, F, wk.WK_BF16, 0.25, batch=b, head_mode=head_mode, ratio_kind=wk.WK_RATIO_NONANCHOR,
                                     score_algo=wk.WK_SCORE_GEMM)
        idx = torch.full((b, G, n_out), -1, dtype=torch.int32, device=d)
        out = [torch.full((b * H * n_out + guard, 128), 7.0, dtype=torch.bfloat16, device=d) for _ in range(2)]
        ws = torch.empty(wk.wk_compress_workspace_bytes(desc), dtype=torch.uint8, device=d)
        wk.wk_compress_chunk(desc, K, V, None, idx, *(x[:b * H * n_out].view(b, H, n_out, 128) for x in out), ws)
        return idx, out, ws[:b * G * (F - 1) * T * 8].view(torch.float64).view(b, G, -1)

    idx, out, scores = call(K, V, 64)
    rows = idx.long().expand(B, H, n_out).unsqueeze(-1).expand(B, H, n_out, 128)
    assert torch.equal(idx[..., :T], torch.arange(T, dtype=torch.int32, device=d).expand(B, G, T))
    for src, got in zip((K, V), out):
        assert torch.equal(got[:B * H * n_out].view(B, H, n_out, 128), torch.gather(src, 2, rows))
        assert (got[B * H * n_out:] == 7.0).all()
    # the lowest scores, the lower index where they tie, in ascending order
    kept = torch.sort(scores, dim=-1, stable=True).indices[..., :n_out - T].sort(dim=-1).values
    assert torch.equal(idx[..., T:], (kept + T).to(torch.int32))
    if F > 1:
        for b in (0, B - 1):
            _, _, one = call(K[b:b + 1].contiguous(), V[b:b + 1].contiguous(), 0)
            # other head ranges: fp32 partial sums in another order
            assert (scores[b] - one[0]).abs().max().item() <= 1e-6
