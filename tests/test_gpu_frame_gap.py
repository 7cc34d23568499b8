"""The frame mask as windows that leave rows out (k_attn_bf16<.., GAP>): the tile with the first row behind the gap wherever it can
fall -- in front of the hand-scheduled loop, at each step of it, behind it --, at both ends of a tile, and windows that the device ends where
the gap does (no window may end earlier) or behind it.  Against the oracle, with the bounds of bf16 attention."""
import importlib.util
import os

import numpy as np
import pytest
import torch

import oracle
import paper_2605_22718_amd as wk
from wkt import K128_PAIR, K256, TWO_RANGES, assert_attention_close_bf16, dev, frame_mask_plan

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_22718_amd", "csrc")


def test_gap_loops_are_what_their_generator_writes():
    spec = importlib.util.spec_from_file_location("gen_attn_loop", os.path.join(CSRC, "gen_attn_loop.py"))
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    for kg, name in gen.GAP_FILES.items():
        assert gen.render(kg, True) == open(os.path.join(CSRC, name)).read()
        # beside the tile loads: the plain loop, instruction for instruction
        def rest(gap):
            return [ln for ln in gen.generate(kg, gap) if ln.startswith(("v_mfma", "v_exp", "v_fma", "v_dot2c", "ds_", "s_waitcnt", "s_barrier"))]
        assert rest(True) == rest(False)


def _check(H, T, F, row0, n_after, n_dev, plan):
    N_q, N_kv, d = F * T, row0 + F * T + n_after, dev()
    assert frame_mask_plan(H, N_q, N_kv, row0, T) == plan
    g = torch.Generator().manual_seed(H + T + row0 + n_after)
    Q, K, V = (torch.randn(H, n, 128, generator=g).to(torch.bfloat16) for n in (N_q, N_kv, N_kv))
    O, lse = torch.full_like(Q, float("nan"), device=d), torch.full(Q.shape[:2], float("nan"), device=d)
    ws = torch.empty(wk.wk_attention_block_causal_workspace_bytes(H, N_q), dtype=torch.uint8, device=d)
    n = None if n_dev is None else torch.tensor([n_dev], dtype=torch.int32, device=d)
    wk.wk_attention_block_causal(Q.to(d), K.to(d), V.to(d), O, row0, T, ws, lse=lse, n_kv_dev=n)
    rows = np.arange(N_q, dtype=np.int32) if H < 10 else np.unique([f * T + r for f in range(F) for r in (0, T // 2, T - 1)]).astype(np.int32)
    ref, ref_lse = oracle.attention_block_causal(Q, K, V, row0, T, N_kv=n_dev, rows=rows, want_lse=True)
    sel = torch.as_tensor(rows, dtype=torch.long)
    assert_attention_close_bf16(O.cpu()[:, sel], ref, lse.cpu()[:, sel], ref_lse)
    assert torch.isfinite(O.float()).all()


# pairs: the gap begins at row row0 + T; tiles 2 .. 15 of windows of 17 and more, and the ends of a tile
@pytest.mark.gpu
@pytest.mark.parametrize("row0", [0, 63, 64, 127, 128, 129, 192, 256, 320, 383, 384, 448, 512, 577, 703, 830])
def test_pairs_with_the_gap_at_every_step(row0):
    _check(30, 130, 2, row0, max(1, 830 - row0), None, K128_PAIR)


@pytest.mark.gpu
@pytest.mark.parametrize("row0", [0, 62, 63, 126, 127, 128, 191, 255, 319, 383, 447, 511, 575, 700])
def test_large_workgroups_with_the_gap_at_every_step(row0):
    _check(64, 129, 3, row0, max(64, 700 - row0), None, K256)


# three frames and one, a last frame without a gap, windows that the device cuts at the chunk's end, one key behind it and inside a tile;
# frames of one token; nothing behind the chunk
@pytest.mark.gpu
@pytest.mark.parametrize("H,T,F,row0,n_after,n_dev,plan", [
    (2, 250, 3, 0, 0, None, K128_PAIR), (3, 249, 3, 130, 191, 130 + 747, K128_PAIR), (3, 249, 3, 130, 191, 130 + 747 + 1, K128_PAIR),
    (5, 333, 2, 63, 1, None, K128_PAIR), (48, 300, 3, 70, 300, 70 + 900 + 77, K128_PAIR), (64, 130, 3, 130, 300, 130 + 390 + 129, K256),
    (64, 130, 3, 130, 191, 130 + 390, K256), (2, 1, 5, 40, 9, None, K256), (70, 65, 1, 3, 300, None, K128_PAIR)])
def test_gaps_and_device_side_lengths(H, T, F, row0, n_after, n_dev, plan):
    _check(H, T, F, row0, n_after, n_dev, plan)


# where two ranges stay the better form
@pytest.mark.gpu
@pytest.mark.parametrize("H,T,F,row0,n_after,plan", [(6, 162, 3, 324, 567, TWO_RANGES + K128_PAIR), (2, 70, 3, 1000, 2000, TWO_RANGES + K128_PAIR),
                                                     (61, 19, 7, 57, 367, TWO_RANGES + K256)])
def test_two_ranges(H, T, F, row0, n_after, plan):
    _check(H, T, F, row0, n_after, None, plan)
