"""Attention over windows that hold infinities: a value of a visible key may be infinite, a key's score may be -inf (weight 0).
What a launch only repeats or pads with -- a range counted twice, a row behind the window's end -- has no part in the result."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_22718_amd as wk
from wkt import ATT_MAX_ABS_F32, assert_attention_close_bf16, attention_errors, dev

pytestmark = pytest.mark.gpu
DTYPES = [torch.bfloat16, torch.float32]
FEATURE = 37


def _inputs(H, N_q, N_kv, dtype, seed):
    g = torch.Generator().manual_seed(seed)
    return [torch.randn(H, n, 128, generator=g).to(dtype) for n in (N_q, N_kv, N_kv)]


def _run(Q, K, V, split):
    d, H, N_q, N_kv = dev(), Q.shape[0], Q.shape[1], K.shape[1]
    n = wk.wk_attention_workspace_bytes(H, N_q, N_kv, wk.WK_BF16 if Q.dtype == torch.bfloat16 else wk.WK_F32) if split else 0
    assert (n > 0) == split
    O, lse = torch.empty_like(Q, device=d), torch.empty(Q.shape[:2], device=d)
    wk.wk_attention(Q.to(d), K.to(d), V.to(d), O, lse, workspace=torch.empty(n, dtype=torch.uint8, device=d) if split else None)
    return O.cpu(), lse.cpu()


def _check(O, lse, Q, K, V):
    ref, ref_lse = oracle.attention(Q, K, V, want_lse=True)
    if Q.dtype == torch.bfloat16:
        assert_attention_close_bf16(O, ref, lse, ref_lse)
    else:
        assert attention_errors(O, ref)[0] <= ATT_MAX_ABS_F32 and np.abs(lse.numpy() - ref_lse).max() <= 1e-4


def _check_infinite_value(Q, K, V, key, split):
    """An infinite value makes one output feature infinite and leaves the others what they are without it."""
    V = V.clone()
    V[:, key, FEATURE] = float("inf")
    O, lse = _run(Q, K, V, split)
    assert (O[..., FEATURE] == float("inf")).all()
    O[..., FEATURE], V[..., FEATURE] = 0, 0
    _check(O, lse, Q, K, V)


# the merge works on four ranges at a time and fills up with the last one
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("H,N_q,N_kv", [(1, 64, 4000), (2, 300, 3000), (1, 33, 4096)])
def test_infinite_value_in_the_last_key_range(H, N_q, N_kv, dtype):
    _check_infinite_value(*_inputs(H, N_q, N_kv, dtype, N_kv), N_kv - 1 - N_kv % 64, split=True)


# key ranges none of whose keys has any weight: their partial results are left out, whatever they hold
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("H,N_q,N_kv", [(1, 64, 4000), (2, 300, 3000)])
def test_key_ranges_without_weight(H, N_q, N_kv, dtype):
    Q, K, V = _inputs(H, N_q, N_kv, dtype, N_kv + 1)
    Q[..., 0] = 1
    K[:, 100:, 0] = float("-inf")
    O, lse = _run(Q, K, V, split=True)
    _check(O, lse, Q, K[:, :100].contiguous(), V[:, :100].contiguous())


# the rows that fill the last fp32 tile of a window
@pytest.mark.parametrize("N_kv", [1, 31, 33, 95, 161])
def test_infinite_value_in_the_last_row_f32(N_kv):
    _check_infinite_value(*_inputs(2, 70, N_kv, torch.float32, N_kv), N_kv - 1, split=False)


# an odd count of whole tiles leaves the second wave group of a 128-query workgroup without one; in a split window the rows
# behind its range are the next range's, whose values have their weight there alone
@pytest.mark.parametrize("split,N_q,N_kv", [(False, 300, 64 * 21), (False, 300, 64 * 9), (True, 300, 64 * 47), (True, 64, 64 * 83)])
def test_infinite_value_beside_an_odd_count_of_tiles(split, N_q, N_kv):
    _check_infinite_value(*_inputs(2, N_q, N_kv, torch.bfloat16, N_kv), N_kv - 1, split=split)


def test_infinite_value_beside_an_odd_count_of_tiles_in_place():
    Q, K, V = _inputs(2, 200, 64 * 11, torch.bfloat16, 5)
    V[:, -1, FEATURE] = float("inf")
    d, cut = dev(), 64 * 6
    store = wk.Store([K[:, cut:].contiguous().to(d)], [V[:, cut:].contiguous().to(d)])
    O, lse = torch.empty_like(Q, device=d), torch.empty(Q.shape[:2], device=d)
    wk.wk_attention_in_place(Q.to(d), K[:, :cut].contiguous().to(d), V[:, :cut].contiguous().to(d), cut, store.desc,
                             torch.zeros(1, dtype=torch.int32, device=d), None, 1, O, lse)
    O, lse = O.cpu(), lse.cpu()
    assert (O[..., FEATURE] == float("inf")).all()
    O[..., FEATURE], V[..., FEATURE] = 0, 0
    _check(O, lse, Q, K, V)


# whole tiles without weight, wherever a wave group or a key range begins with one: every other tile of 32 or 64 keys, and
# all but the last
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("H,N_q,N_kv,split", [(2, 200, 160, False), (2, 300, 700, False), (2, 300, 3000, True), (1, 64, 4000, True)])
@pytest.mark.parametrize("tile,skip", [(32, 1), (64, 1), (64, 0)])
def test_tiles_without_weight(H, N_q, N_kv, split, tile, skip, dtype):
    Q, K, V = _inputs(H, N_q, N_kv, dtype, N_kv + tile)
    Q[..., 0] = 1
    dead = (torch.arange(N_kv) // tile) % 2 == skip
    K[:, dead, 0] = float("-inf")
    O, lse = _run(Q, K, V, split)
    _check(O, lse, Q, K[:, ~dead].contiguous(), V[:, ~dead].contiguous())
