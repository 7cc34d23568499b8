"""bf16 attention in each layout of a launch -- 256-query workgroups, 128-query workgroups whose two wave groups take the
even and the odd key tiles, 128-query workgroups of four waves -- and the first two with a split key range.  Which
layout a shape takes is pinned: a change of the library's choice must not leave one untested."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_22718_amd as wk
from wkt import (ATT_MAX_ABS_F32, K128, K128_PAIR, K256, TWO_RANGES, assert_attention_close_bf16, attention_errors, attention_plan, dev,
                 frame_mask_plan)

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


def _device_int(n):
    return None if n is None else torch.tensor([n], dtype=torch.int32, device=dev())


def _check_rows(Q, K, V, O, lse, rows=(0, 31, 32, 255, 256, 700, -1)):
    """Sampled rows of a launch with many queries, against the oracle."""
    rows = np.unique([r % Q.shape[1] for r in rows]).astype(np.int32)
    ref, ref_lse = oracle.attention(Q, K, V, rows=rows, want_lse=True)
    sel = torch.as_tensor(rows, dtype=torch.long)
    assert not torch.isnan(O.float()).any() and not torch.isnan(lse).any()
    assert_attention_close_bf16(O[:, sel.to(O.device)], ref, lse[:, sel.to(lse.device)], ref_lse)


# 128-query workgroups: one tile (a second wave group has none), one partial tile, one pair, an odd tile behind whole pairs,
# a last pair whose second tile is partial / whose first tile is, trips of the steady loop with 0 and 1 left-over steps.
# With N_kv as the window's length the short ones run in four waves; as a length on the device they all run in pairs.
@pytest.mark.parametrize("N_q", [1, 128, 129, 300])
@pytest.mark.parametrize("n_dev", [1, 63, 64, 65, 128, 129, 191, 192, 320, 400, 576, 640, 707])
def test_tile_pairs_by_device_length(N_q, n_dev):
    assert attention_plan(2, N_q, 900) == (K128_PAIR, 1)
    Q, K, V = _inputs(2, N_q, 900, seed=N_q * 1000 + n_dev)
    d = dev()
    O, lse = torch.empty_like(Q, device=d), torch.empty(Q.shape[:2], device=d)
    wk.wk_attention(Q.to(d), K.to(d), V.to(d), O, lse, n_kv_dev=_device_int(n_dev))
    ref, ref_lse = oracle.attention(Q, K, V, N_kv=n_dev, want_lse=True)
    assert_attention_close_bf16(O, ref, lse, ref_lse)


@pytest.mark.parametrize("N_kv,layout", [(1, K128), (64, K128), (65, K128), (129, K128), (200, K128), (320, K128), (449, K128_PAIR)])
def test_small_grids_of_short_windows(N_kv, layout):
    H, N_q, d = 3, 257, dev()
    assert attention_plan(H, N_q, N_kv) == (layout, 1)
    Q, K, V = _inputs(H, N_q, N_kv, seed=N_kv)
    O, lse = torch.empty_like(Q, device=d), torch.empty(Q.shape[:2], device=d)
    wk.wk_attention(Q.to(d), K.to(d), V.to(d), O, lse)
    ref, ref_lse = oracle.attention(Q, K, V, want_lse=True)
    assert_attention_close_bf16(O, ref, lse, ref_lse)


# 256-query workgroups: 1 to 15 tiles, whole and ragged, by the window's length and by a length on the device
@pytest.mark.parametrize("N_kv,n_dev", [(1, None), (63, None), (64, None), (65, None), (200, None), (320, None), (449, None), (577, None),
                                        (707, None), (900, None), (900, 1), (900, 64), (900, 130), (900, 705)])
def test_large_grids(N_kv, n_dev):
    H, N_q, d = 40, 1100, dev()
    assert attention_plan(H, N_q, N_kv) == (K256, 1)
    Q, K, V = _inputs(H, N_q, N_kv, seed=N_kv)
    O, lse = torch.empty_like(Q, device=d), torch.empty(Q.shape[:2], device=d)
    wk.wk_attention(Q.to(d), K.to(d), V.to(d), O, lse, n_kv_dev=_device_int(n_dev))
    _check_rows(Q, K[:, :n_dev].contiguous(), V[:, :n_dev].contiguous(), O, lse)


# 256-query workgroups with a split key range: whole, ending inside a range, and with ranges that are empty
@pytest.mark.parametrize("n_dev", [None, 3601, 1700, 100])
def test_split_large_workgroups(n_dev):
    H, N_q, N_kv, d = 40, 512, 5200, dev()
    n = wk.wk_attention_workspace_bytes(H, N_q, N_kv, wk.WK_BF16)
    layout, splits = attention_plan(H, N_q, N_kv, n)
    assert layout == K256 and splits > 1
    Q, K, V = _inputs(H, N_q, N_kv, seed=9)
    O, lse = torch.empty_like(Q, device=d), torch.empty(Q.shape[:2], device=d)
    wk.wk_attention(Q.to(d), K.to(d), V.to(d), O, lse, workspace=torch.empty(n, dtype=torch.uint8, device=d), n_kv_dev=_device_int(n_dev))
    _check_rows(Q, K[:, :n_dev].contiguous(), V[:, :n_dev].contiguous(), O, lse, rows=(0, 32, 255, 256, -1))


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
    assert torch.equal(lse, only)   # even and odd tiles are summed apart by every layout; no maximum here moves after the first tile


@pytest.mark.parametrize("N_kv", [640, 1500, 2111])
def test_tile_pairs_with_rising_logits(N_kv):
    Q, K, V = _inputs(2, 200, N_kv, seed=N_kv, rising=True)
    d = dev()
    O, lse = torch.empty_like(Q, device=d), torch.empty(Q.shape[:2], device=d)
    only = torch.empty_like(lse)
    wk.wk_attention(Q.to(d), K.to(d), V.to(d), O, lse)
    wk.wk_attention(Q.to(d), K.to(d), None, None, only)
    ref, ref_lse = oracle.attention(Q, K, V, want_lse=True)
    assert_attention_close_bf16(O, ref, lse, ref_lse)
    # the groups' maxima move at other tiles than those of a wave that walks them all: every weight is rounded to bf16 against
    # another maximum.  bf16 has 8 significant bits: half a unit in the last place is 2^-8 of the weight at most, on either side,
    # so the sums differ by 2^-7 of them at most (one weight can be all of a sum), and by their fp32 rounding
    assert (lse - only).abs().max().item() <= 2.0 ** -7 + 1e-5
    assert np.abs(only.cpu().numpy() - ref_lse).max() <= 2e-2


# splits whose tile counts are odd (the second group's last tile belongs to the next split), end past the device-side
# length, or are empty
@pytest.mark.parametrize("H,N_q,N_kv,n_dev", [(2, 300, 3000, None), (2, 231, 6001, None), (4, 537, 2975, 1700), (1, 65, 5000, 130)])
def test_split_tile_pairs(H, N_q, N_kv, n_dev):
    Q, K, V = _inputs(H, N_q, N_kv, seed=N_kv + N_q)
    d = dev()
    n = wk.wk_attention_workspace_bytes(H, N_q, N_kv, wk.WK_BF16)
    layout, splits = attention_plan(H, N_q, N_kv, n)
    assert layout == K128_PAIR and splits > 1
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
@pytest.mark.parametrize("capacity", [0, 16])   # chunks the call could have listed: with 16 the host expects a window long enough for pairs
def test_tile_pairs_in_place(n_native, lens, capacity):
    H, N_q, d = 2, 150, dev()
    g = torch.Generator().manual_seed(n_native + len(lens))
    Q = torch.randn(H, N_q, 128, generator=g).to(torch.bfloat16)
    parts = [tuple(torch.randn(H, n, 128, generator=g).to(torch.bfloat16) for _ in range(2)) for n in [n_native] + lens]
    store = wk.Store(*[[p[i].to(d) for p in (parts[1:] or parts[:1])] for i in range(2)])
    R = max(len(lens), capacity if lens else 0)
    longest = n_native + R * max(lens, default=0)
    assert attention_plan(H, N_q, max(64, longest))[0] == (K128_PAIR if longest > 352 else K128)
    O, lse = torch.empty_like(Q, device=d), torch.empty(Q.shape[:2], device=d)
    ids = torch.arange(R, dtype=torch.int32, device=d) if lens else None
    wk.wk_attention_in_place(Q.to(d), parts[0][0].to(d) if n_native else None, parts[0][1].to(d) if n_native else None, n_native,
                             store.desc, ids, _device_int(len(lens)) if lens else None, R, O, lse)
    K, V = (torch.cat([p[i] for p in parts], 1) for i in range(2))
    ref, ref_lse = oracle.attention(Q, K, V, want_lse=True)
    assert_attention_close_bf16(O, ref, lse, ref_lse)


# in place with 256-query workgroups: unequal chunks, a segment of one key, ids that are skipped, a window of one tile
@pytest.mark.parametrize("n_native,lens,ids", [(200, [64, 1, 130], [2, -1, 0, 99, 1]), (0, [40, 3, 3], [0]), (131, [1, 63, 500], [1, 0, 2]), (65, [7, 7, 7], [5])])
def test_large_grids_in_place(n_native, lens, ids):
    H, N_q, d = 40, 1100, dev()
    assert attention_plan(H, N_q, max(64, n_native + len(ids) * max(lens)))[0] == K256
    g = torch.Generator().manual_seed(n_native)
    Q = torch.randn(H, N_q, 128, generator=g).to(torch.bfloat16)
    parts = [tuple(torch.randn(H, n, 128, generator=g).to(torch.bfloat16) for _ in range(2)) for n in [n_native] + lens]
    store = wk.Store(*[[p[i].to(d) for p in parts[1:]] for i in range(2)])
    O, lse = torch.empty_like(Q, device=d), torch.empty(Q.shape[:2], device=d)
    wk.wk_attention_in_place(Q.to(d), parts[0][0].to(d) if n_native else None, parts[0][1].to(d) if n_native else None, n_native,
                             store.desc, torch.tensor(ids, dtype=torch.int32, device=d), None, len(ids), O, lse)
    window = [parts[0]] + [parts[1 + i] for i in ids if 0 <= i < len(lens)]
    _check_rows(Q, *(torch.cat([p[i] for p in window], 1) for i in range(2)), O, lse)


# the frame mask's tables of launches, windows with a gap and two key ranges, each in 128-query workgroups (small grids) and in 256-query
# ones: frames that end inside a query tile; behind the chunk an odd count of tiles, one key, no key, by the host's length and by the device's
@pytest.mark.parametrize("H,T,F,row0,n_after,n_dev,plan", [
    (2, 250, 3, 0, 0, None, K128_PAIR), (2, 129, 3, 64, 1, None, K128_PAIR), (3, 249, 3, 130, 191, None, K128_PAIR), (48, 300, 3, 0, 0, None, K128_PAIR),
    (48, 300, 3, 70, 1, None, K128_PAIR), (48, 300, 3, 70, 300, 70 + 900, K128_PAIR), (64, 130, 3, 130, 191, None, K256),
    (64, 130, 3, 130, 300, 130 + 390 + 1, K256),
    (39, 21, 7, 847, 0, None, TWO_RANGES + K128_PAIR), (44, 22, 6, 918, 1, None, TWO_RANGES + K128_PAIR), (6, 162, 3, 324, 567, None, TWO_RANGES + K128_PAIR),
    (6, 162, 3, 324, 567, 324 + 486, TWO_RANGES + K128_PAIR), (6, 162, 3, 324, 567, 324 + 486 + 1, TWO_RANGES + K128_PAIR),
    (44, 129, 6, 685, 0, None, TWO_RANGES + K256), (57, 129, 5, 862, 1, None, TWO_RANGES + K256), (47, 132, 3, 483, 648, None, TWO_RANGES + K256),
    (47, 132, 3, 483, 648, 483 + 396, TWO_RANGES + K256), (47, 132, 3, 483, 648, 483 + 396 + 1, TWO_RANGES + K256)])
def test_frame_mask_layouts(H, T, F, row0, n_after, n_dev, plan):
    N_q, d = F * T, dev()
    assert frame_mask_plan(H, N_q, row0 + N_q + n_after, row0, T) == plan
    Q, K, V = _inputs(H, N_q, row0 + N_q + n_after, seed=T + H)
    O, lse = torch.empty_like(Q, device=d), torch.empty(Q.shape[:2], device=d)
    ws = torch.empty(wk.wk_attention_block_causal_workspace_bytes(H, N_q), dtype=torch.uint8, device=d)
    wk.wk_attention_block_causal(Q.to(d), K.to(d), V.to(d), O, row0, T, ws, lse=lse, n_kv_dev=_device_int(n_dev))
    rows = np.arange(N_q, dtype=np.int32) if H < 10 else np.unique([r for r in (0, T - 1, T, 2 * T - 1, 2 * T, 255, 256, N_q - 1) if r < N_q]).astype(np.int32)
    ref, ref_lse = oracle.attention_block_causal(Q, K, V, row0, T, N_kv=n_dev, rows=rows, want_lse=True)
    sel = torch.as_tensor(rows, dtype=torch.long)
    assert_attention_close_bf16(O.cpu()[:, sel], ref, lse.cpu()[:, sel], ref_lse)
