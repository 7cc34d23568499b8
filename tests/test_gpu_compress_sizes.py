"""Scores, selection and rows of wk_compress_chunk at the edges of its passes: lists over one to three heads, over more heads than a
workgroup holds the mean of, tokens that leave waves and lane groups without one, and chunks past the caches, whose passes stream."""
import pytest
import torch

import paper_2605_22718_amd as wk
from wkt import dev

pytestmark = pytest.mark.gpu
SHARED, PER_HEAD = wk.WK_HEADS_SHARED, wk.WK_HEADS_INDEPENDENT


@pytest.mark.parametrize("dtype,heads,B,H,T,F", [
    (torch.bfloat16, SHARED, 1, 1, 5, 2), (torch.bfloat16, SHARED, 2, 3, 33, 3), (torch.float32, SHARED, 1, 2, 17, 2),
    (torch.bfloat16, SHARED, 1, 4, 9, 3), (torch.float32, SHARED, 3, 21, 12, 2), (torch.bfloat16, SHARED, 2, 41, 13, 2),
    (torch.bfloat16, SHARED, 1, 64, 8, 2), (torch.bfloat16, SHARED, 2, 65, 11, 2), (torch.float32, SHARED, 1, 130, 7, 3),
    (torch.bfloat16, PER_HEAD, 2, 5, 1, 2), (torch.float32, PER_HEAD, 1, 3, 65, 2),
    # K beyond 64 MiB (bf16) and 144 MiB (fp32)
    (torch.bfloat16, SHARED, 3, 65, 1001, 2), (torch.bfloat16, SHARED, 9, 3, 3501, 3), (torch.bfloat16, PER_HEAD, 5, 7, 2731, 3),
    (torch.float32, SHARED, 5, 5, 4100, 3), (torch.float32, PER_HEAD, 3, 11, 3203, 3)])
def test_against_fp64(dtype, heads, B, H, T, F):
    d = dev()
    g = torch.Generator(device=d).manual_seed(1000 * H + T)
    K, V = (torch.randn((B, H, F * T, 128), generator=g, device=d).to(dtype) for _ in range(2))
    G = H if heads == PER_HEAD else 1
    desc = wk.make_compress_desc(H, T, F, wk.WK_F32 if dtype == torch.float32 else wk.WK_BF16, 0.5, batch=B, head_mode=heads,
                                 ratio_kind=wk.WK_RATIO_NONANCHOR)
    n_out, _ = wk.wk_keep_count(0.5, wk.WK_RATIO_NONANCHOR, wk.WK_ANCHOR_FIRST_FRAME, F, T)
    idx = torch.full((B, G, n_out), -1, dtype=torch.int32, device=d)
    guard = 64
    out = [torch.full((B * H * n_out + guard, 128), 7.0, dtype=dtype, device=d) for _ in range(2)]
    ws = torch.empty(wk.wk_compress_workspace_bytes(desc), dtype=torch.uint8, device=d)
    wk.wk_compress_chunk(desc, K, V, None, idx, *(x[:B * H * n_out].view(B, H, n_out, 128) for x in out), ws)
    scores = ws[:B * G * (F - 1) * T * 8].view(torch.float64).view(B, G, -1)
    for b in range(B):   # Eq. 5 in its factored form; a list's vectors span its heads
        k = K[b].double().view(G, H // G, F * T, 128).transpose(1, 2).reshape(G, F * T, -1)
        unit = k / k.norm(dim=-1, keepdim=True)
        want = (unit[:, T:] * unit[:, :T].mean(1, keepdim=True)).sum(-1)
        assert (scores[b] - want).abs().max().item() <= 1e-7   # fp32 sums of 8 products and a mean rounded to fp32 (measured 4e-10)
    kept = torch.sort(scores, dim=-1, stable=True).indices[..., :n_out - T].sort(dim=-1).values
    assert torch.equal(idx[..., :T], torch.arange(T, dtype=torch.int32, device=d).expand(B, G, T))
    assert torch.equal(idx[..., T:], (kept + T).to(torch.int32))
    rows = idx.long().expand(B, H, n_out).unsqueeze(-1).expand(B, H, n_out, 128)
    for src, got in zip((K, V), out):
        assert torch.equal(got[:B * H * n_out].view(B, H, n_out, 128), torch.gather(src, 2, rows))
        assert (got[B * H * n_out:] == 7.0).all()


# the anchors' norms with the partial means (few rows and heads) or before them, the mean folded by the score kernel (few partial sums) or before it: each
# alone, both and neither, with tokens and heads that fill no whole batch of loads
@pytest.mark.parametrize("dtype,heads,B,H,T,F", [
    (torch.bfloat16, SHARED, 1, 8, 499, 3), (torch.bfloat16, SHARED, 1, 8, 651, 2), (torch.bfloat16, SHARED, 1, 9, 301, 2), (torch.bfloat16, SHARED, 1, 9, 701, 2),
    (torch.float32, SHARED, 2, 7, 67, 3), (torch.float32, SHARED, 1, 5, 33, 2), (torch.bfloat16, SHARED, 3, 2, 129, 2), (torch.float32, SHARED, 1, 3, 1, 2),
    (torch.bfloat16, PER_HEAD, 1, 11, 1013, 3), (torch.float32, PER_HEAD, 2, 3, 64, 2), (torch.bfloat16, PER_HEAD, 8, 8, 1000, 3)])
def test_launches_saved(dtype, heads, B, H, T, F):
    test_against_fp64(dtype, heads, B, H, T, F)


# either side of the bounds behind which the mean is folded by a launch of its own
@pytest.mark.parametrize("dtype,heads,B,H,T,F", [
    (torch.bfloat16, PER_HEAD, 1, 32, 1024, 2), (torch.bfloat16, PER_HEAD, 1, 34, 960, 2), (torch.bfloat16, PER_HEAD, 1, 35, 960, 2),
    (torch.bfloat16, PER_HEAD, 1, 64, 1024, 2), (torch.bfloat16, PER_HEAD, 1, 65, 1024, 2), (torch.bfloat16, SHARED, 1, 4, 1584, 2), (torch.bfloat16, SHARED, 1, 4, 1585, 2)])
def test_mean_fold_bounds(dtype, heads, B, H, T, F):
    test_against_fp64(dtype, heads, B, H, T, F)
