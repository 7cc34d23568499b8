"""bf16 attention in each layout of a launch: 256-query workgroups, 128-query workgroups whose two wave groups take the
even and the odd key tiles, and either with a split key range."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_22718_amd as wk
from wkt import ATT_MAX_ABS_F32, assert_attention_close_bf16, attention_errors, dev

pytestmark = pytest.mark.gpu


def _assert_close_f32(O, lse, ref, ref_lse, tol=ATT_MAX_ABS_F32):
    assert attention_errors(O, ref)[0] <= tol and np.abs(lse.cpu().numpy() - ref_lse).max() <= 1e-4


def _inputs(H, N_q, N_kv, seed, rising=False):
    g = torch.Generator().manual_seed(seed)
    Q, K, V = (torch.randn(H, n, 128, generator=g).to(torch.bfloat16) for n in (N_q, N_kv, N_kv))
    if rising:   # later keys have larger logits: the running maximum moves in every tile, in both wave groups
        Q = (Q.float() * 6).to(torch.bfloat16)
        order = torch.argsort((Q[:, :1].float() @ K.float().transpose(1, 2))[:, 0], dim=1)
        K = torch.stack([K[h, order[h]] for h in range(H)])
    return Q, K, V


# 128-query workgroups: one tile (the second group has none), one partial tile, one pair, an odd tile behind whole pairs,
# a last pair whose second tile is partial / whose first tile is, trips of the steady loop with 0 and 1 left-over steps
@pytest.mark.parametrize("N_q", [1, 127, 128, 129, 300])
@pytest.mark.parametrize("N_kv", [1, 63, 64, 65, 128, 129, 191, 192, 320, 400, 576, 640, 707])
def test_tile_pairs(N_q, N_kv):
    Q, K, V = _inputs(2, N_q, N_kv, seed=N_q * 1000 + N_kv)
    d = dev()
    O, lse = torch.empty_like(Q, device=d), torch.empty(Q.shape[:2], device=d)
    only = torch.empty_like(lse)
    wk.wk_attention(Q.to(d), K.to(d), V.to(d), O, lse)
    wk.wk_attention(Q.to(d), K.to(d), None, None, only)
    ref, ref_lse = oracle.attention(Q, K, V, want_lse=True)
    assert_attention_close_bf16(O, ref, lse, ref_lse)
    assert torch.equal(lse, only)   # the row sums do not depend on which kernel or layout forms them


@pytest.mark.parametrize("N_kv", [640, 1500, 2111])
def test_tile_pairs_with_rising_logits(N_kv):
    Q, K, V = _inputs(2, 200, N_kv, seed=N_kv, rising=True)
    d = dev()
    O, lse = torch.empty_like(Q, device=d), torch.empty(Q.shape[:2], device=d)
    wk.wk_attention(Q.to(d), K.to(d), V.to(d), O, lse)
    ref, ref_lse = oracle.attention(Q, K, V, want_lse=True)
    assert_attention_close_bf16(O, ref, lse, ref_lse)


# splits whose tile counts are odd (the second group's last tile belongs to the next split), end past the device-side
# length, or are empty
@pytest.mark.parametrize("H,N_q,N_kv,n_dev", [(2, 300, 3000, None), (2, 231, 6001, None), (4, 537, 2975, 1700), (1, 65, 5000, 130)])
def test_split_tile_pairs(H, N_q, N_kv, n_dev):
    Q, K, V = _inputs(H, N_q, N_kv, seed=N_kv + N_q)
    d = dev()
    n = wk.wk_attention_workspace_bytes(H, N_q, N_kv, wk.WK_BF16)
    assert n > 0
    O, lse = torch.empty_like(Q, device=d), torch.empty(Q.shape[:2], device=d)
    wk.wk_attention(Q.to(d), K.to(d), V.to(d), O, lse, workspace=torch.empty(n, dtype=torch.uint8, device=d),
                    n_kv_dev=None if n_dev is None else torch.tensor([n_dev], dtype=torch.int32, device=d))
    ref, ref_lse = oracle.attention(Q, K, V, N_kv=n_dev or N_kv, want_lse=True)
    assert_attention_close_bf16(O, ref, lse, ref_lse)


# fp32, pairs of 32-key tiles: one tile (the second wave group has none), one key, a partial first and second tile of a
# pair, odd and even counts; queries that leave waves of a workgroup without one
@pytest.mark.parametrize("N_q", [1, 32, 33, 128, 161])
@pytest.mark.parametrize("N_kv", [1, 31, 32, 33, 64, 65, 95, 97, 128, 161])
def test_tile_pairs_f32(N_q, N_kv):
    Q, K, V = (x.float() for x in _inputs(2, N_q, N_kv, seed=N_q * 1000 + N_kv))
    d = dev()
    O, lse = torch.empty_like(Q, device=d), torch.empty(Q.shape[:2], device=d)
    only = torch.empty_like(lse)
    wk.wk_attention(Q.to(d), K.to(d), V.to(d), O, lse)
    wk.wk_attention(Q.to(d), K.to(d), None, None, only)
    ref, ref_lse = oracle.attention(Q, K, V, want_lse=True)
    _assert_close_f32(O, lse, ref, ref_lse)
    assert torch.equal(lse, only)


# 2e-4: logits six times as large, see the large-logit case of test_gpu_attention.py
@pytest.mark.parametrize("rising,tol", [(False, ATT_MAX_ABS_F32), (True, 2e-4)])
@pytest.mark.parametrize("H,N_q,N_kv,n_dev", [(2, 300, 1500, None), (1, 65, 3001, 517), (3, 129, 2000, 40)])
def test_split_tile_pairs_f32(H, N_q, N_kv, n_dev, rising, tol):
    Q, K, V = (x.float() for x in _inputs(H, N_q, N_kv, seed=N_kv + N_q, rising=rising))
    d = dev()
    n = wk.wk_attention_workspace_bytes(H, N_q, N_kv, wk.WK_F32)
    assert n > 0
    O, lse = torch.empty_like(Q, device=d), torch.empty(Q.shape[:2], device=d)
    wk.wk_attention(Q.to(d), K.to(d), V.to(d), O, lse, workspace=torch.empty(n, dtype=torch.uint8, device=d),
                    n_kv_dev=None if n_dev is None else torch.tensor([n_dev], dtype=torch.int32, device=d))
    ref, ref_lse = oracle.attention(Q, K, V, N_kv=n_dev or N_kv, want_lse=True)
    _assert_close_f32(O, lse, ref, ref_lse, tol)


# in place: odd and even totals of tiles, segments that end inside a tile (the pair then spans two segments), one tile in all
@pytest.mark.parametrize("n_native,lens", [(0, [40]), (64, [64]), (100, [64, 1, 200]), (129, [63, 65, 130, 64]), (300, [])])
def test_tile_pairs_in_place(n_native, lens):
    H, N_q, d = 2, 150, dev()
    g = torch.Generator().manual_seed(n_native + len(lens))
    Q = torch.randn(H, N_q, 128, generator=g).to(torch.bfloat16)
    parts = [tuple(torch.randn(H, n, 128, generator=g).to(torch.bfloat16) for _ in range(2)) for n in [n_native] + lens]
    store = wk.Store(*[[p[i].to(d) for p in (parts[1:] or parts[:1])] for i in range(2)])
    O, lse = torch.empty_like(Q, device=d), torch.empty(Q.shape[:2], device=d)
    ids = torch.arange(len(lens), dtype=torch.int32, device=d) if lens else None
    wk.wk_attention_in_place(Q.to(d), parts[0][0].to(d) if n_native else None, parts[0][1].to(d) if n_native else None, n_native,
                             store.desc, ids, None, len(lens), O, lse)
    K, V = (torch.cat([p[i] for p in parts], 1) for i in range(2))
    ref, ref_lse = oracle.attention(Q, K, V, want_lse=True)
    assert_attention_close_bf16(O, ref, lse, ref_lse)


# the frame mask's table of launches in 128-query workgroups (small grids): frames that end
# inside a query tile, a key range behind the chunk that is empty, one key, and an odd count of tiles
@pytest.mark.parametrize("H,T,row0,n_after", [(2, 250, 0, 0), (2, 129, 64, 1), (3, 249, 130, 191)])
def test_frame_mask_layouts(H, T, row0, n_after):
    N_q, d = 3 * T, dev()
    Q, K, V = _inputs(H, N_q, row0 + N_q + n_after, seed=T + H)
    O, lse = torch.empty_like(Q, device=d), torch.empty(Q.shape[:2], device=d)
    ws = torch.empty(wk.wk_attention_block_causal_workspace_bytes(H, N_q), dtype=torch.uint8, device=d)
    wk.wk_attention_block_causal(Q.to(d), K.to(d), V.to(d), O, row0, T, ws, lse=lse)
    ref, ref_lse = oracle.attention_block_causal(Q, K, V, row0, T, want_lse=True)
    assert_attention_close_bf16(O, ref, lse, ref_lse)
