"""fp32 attention works on two fp16 parts of every number and on powers of two that take them there, found from a workgroup's first
tile of keys; where numbers do not fit, on fp32 products.  Both against the oracle, over scales and at the edges of tiles and wave groups."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_22718_amd as wk
from wkt import ATT_MAX_ABS_F32, dev

pytestmark = pytest.mark.gpu


def _check(Q, K, V, unit, split=False, tol=ATT_MAX_ABS_F32):
    """unit: what the values of a feature are of the size of."""
    d, H, N_q, N_kv = dev(), Q.shape[0], Q.shape[1], K.shape[1]
    n = wk.wk_attention_workspace_bytes(H, N_q, N_kv, wk.WK_F32) if split else 0
    assert (n > 0) == split
    O, lse, only = torch.empty_like(Q, device=d), torch.empty((H, N_q), device=d), torch.empty((H, N_q), device=d)
    wk.wk_attention(Q.to(d), K.to(d), V.to(d), O, lse, workspace=torch.empty(n, dtype=torch.uint8, device=d) if split else None)
    wk.wk_attention(Q.to(d), K.to(d), V.to(d), None, only)
    ref, ref_lse = oracle.attention(Q, K, V, want_lse=True)
    assert np.abs((O.cpu().double().numpy() - ref) / np.asarray(unit)).max() <= tol
    assert np.abs(lse.cpu().double().numpy() - ref_lse).max() <= 1e-5 and np.abs(only.cpu().double().numpy() - ref_lse).max() <= 1e-5


def _randn(H, N_q, N_kv, seed=3):
    g = torch.Generator().manual_seed(seed)
    return [torch.randn(H, n, 128, generator=g) for n in (N_q, N_kv, N_kv)]


# 128 queries a workgroup, one or two tiles of 32 keys a step
@pytest.mark.parametrize("H,N_q,N_kv,split", [(1, 1, 1, False), (2, 33, 31, False), (1, 128, 32, False), (3, 129, 33, False), (2, 70, 64, False), (1, 97, 65, False),
                                             (2, 40, 255, False), (2, 256, 257, True), (300, 5, 65, False), (300, 20, 300, False), (1, 64, 4000, True)])
def test_edges(H, N_q, N_kv, split):
    Q, K, V = _randn(H, N_q, N_kv)
    _check(Q, K, V, 1.0, split)


# the last: no power of two within 2^60
@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("q,k,v", [(1, 1, 1e-12), (1e6, 1e-6, 1e12), (1e-10, 1e10, 3e-5), (1e-25, 1e25, 1e30)])
def test_scales(q, k, v, split):
    Q, K, V = _randn(2, 100, 300)
    Q[:, 7] = 0
    v = v * torch.logspace(-2, 2, 128)   # features of different size
    _check(Q * q, K * k, V * v, np.asarray(v.double()), split)


# tiles that the first one's scales do not fit: larger keys and values, values that become small, a first tile of zeros, one element
@pytest.mark.parametrize("H,N_q,N_kv,split", [(2, 100, 300, False), (2, 100, 300, True), (300, 10, 96, False)])
@pytest.mark.parametrize("case", ["keys", "values", "small", "zeros", "tiny_after_zeros", "one"])
def test_tiles_unlike_the_first(case, H, N_q, N_kv, split):
    Q, K, V = _randn(H, N_q, N_kv)
    unit = 1.0
    if case == "keys":
        K[:, 40:] *= 60
        Q /= 60
    if case == "values":
        V[:, 70:] *= 500
        unit = 500.0
    if case == "small":   # the first rows have no weight, so that the small ones are what is left
        Q[..., 0] = 4
        K[..., 0] = torch.where(torch.arange(N_kv) < 33, -300.0, 0.0)
        V[:, 33:] *= 1e-5
        unit = 1e-5
    if case in ("zeros", "tiny_after_zeros"):
        K[:, :33] = 0
        V[:, :33] = 0
    if case == "tiny_after_zeros":
        V *= 1e-7
        unit = 1e-7
    if case == "one":
        V[0, 50, 3] = 3e4
        K[0, 45, 77] = 200
        Q[..., 77] = 0
        unit = np.where(np.arange(128) == 3, 3e4, 1.0)
    _check(Q, K, V, unit, split)


# One number that sets a power of two for others which it has nothing to do with, and weights or values that are small beside it: the parts alone
# lose them, more with every power of ten.  (20 and 52 keys: one partial tile, and one behind the first; 300: two wave groups, key ranges)
def _unlike(case, x, Q, K, V, at):
    """-> the size of the outputs"""
    at %= K.shape[1]
    first = slice(0, 32 if K.shape[1] > 32 else 10)
    if case == "masked_key":
        Q[..., 0], K[..., 0] = 1, 0
        K[:, at, 0] = -x
    if case == "query_channel":
        Q[..., 7], K[..., 7] = x, 0
    if case == "key_channel":
        Q[..., 7], K[..., 7] = 0, x
    if case == "zeros_then_small":
        K[:, :at] = 0
        K /= x
        Q *= x
    if case in ("large_value", "large_values", "one_feature"):   # without weight: e^-53
        Q[..., 0], K[..., 0] = 1, 0
        K[:, at if case != "large_values" else first, 0] = -600
    if case == "large_value":
        V[:, at] = x
    if case == "large_values":
        V[:, first] *= x
    unit = np.ones(128)
    if case == "one_feature":
        unit[9] = 1e-4
        V[..., 9] *= 1e-4
        V[:, at, 9] = x * 1e-4
    if case == "sink":   # a key without values that takes all but 1 / x of the weight
        Q[..., 0], K[..., 0] = 16, 0
        K[:, at], V[:, at] = 0, 0
        K[:, at, 0] = float(np.float16(np.log(x) / np.sqrt(2)))   # (a logit of one product, exact in parts)
        unit = unit * np.abs(oracle.attention(Q, K, V)).max() / 4
    return unit


@pytest.mark.parametrize("H,N_q,N_kv,split", [(2, 64, 20, False), (3, 33, 52, False), (2, 100, 300, False), (2, 100, 300, True), (300, 10, 96, False)])
@pytest.mark.parametrize("at", [5, 45, 290])
@pytest.mark.parametrize("case,x", [(c, x) for c, xs in (
    ("masked_key", (1e3, 1e4, 1e6, 1e9, 1e12, 1e15)), ("query_channel", (1e4, 1e6, 1e9, 1e12)), ("key_channel", (1e4, 1e9, 1e12)),
    ("zeros_then_small", (1e3, 1e6)), ("large_value", (1e3, 1e6, 1e9, 1e12)), ("large_values", (1e3, 1e6, 1e9)), ("one_feature", (1e3, 1e6)),
    ("sink", (1e2, 1e5, 1e9, 1e13))) for x in xs])
def test_numbers_that_others_are_small_beside(case, x, at, H, N_q, N_kv, split):
    Q, K, V = _randn(H, N_q, N_kv)
    unit = _unlike(case, x, Q, K, V, at)
    _check(Q, K, V, unit, split)


@pytest.mark.parametrize("case,x", [("masked_key", 1e6), ("masked_key", 1e12), ("query_channel", 1e9), ("large_value", 1e9)])
@pytest.mark.parametrize("T,F,row0,N_kv", [(100, 2, 0, 300), (40, 3, 70, 190)])
def test_numbers_that_others_are_small_beside_under_the_frame_mask(case, x, T, F, row0, N_kv):
    d = dev()
    Q, K, V = _randn(2, T * F, N_kv)
    unit = _unlike(case, x, Q, K, V, row0 + 5)
    O, lse = torch.empty_like(Q, device=d), torch.empty((2, T * F), device=d)
    ws = torch.empty(wk.wk_attention_block_causal_workspace_bytes(2, T * F), dtype=torch.uint8, device=d)
    wk.wk_attention_block_causal(Q.to(d), K.to(d), V.to(d), O, row0, T, ws, lse=lse)
    ref, ref_lse = oracle.attention_block_causal(Q, K, V, row0, T, want_lse=True)
    assert np.abs((O.cpu().double().numpy() - ref) / unit).max() <= ATT_MAX_ABS_F32
    assert np.abs(lse.cpu().double().numpy() - ref_lse).max() <= 1e-5


@pytest.mark.parametrize("case,x", [("masked_key", 1e6), ("masked_key", 1e12), ("query_channel", 1e9), ("zeros_then_small", 1e6)])
def test_numbers_that_others_are_small_beside_in_stored_chunks(case, x):
    d = dev()
    Q, K, V = _randn(3, 70, 240)
    _unlike(case, x, Q, K, V, 45)
    Ks = [k.contiguous() for k in K.split([100, 52, 88], 1)]
    store = wk.Store([k.to(d) for k in Ks], [k.to(d) for k in Ks])
    out = torch.empty((3, 3, 70), device=d)
    wk.wk_chunk_lse(store.desc, Q.to(d), out)
    for k, got in zip(Ks, out.cpu().double().numpy()):
        assert np.abs(got - oracle.attention(Q, k, k, want_lse=True)[1]).max() <= 1e-5


# the walk on fp32 products: whole and partial tiles, odd counts of them, known from the first tile (5) or from the last one
@pytest.mark.parametrize("H,N_q", [(2, 130), (300, 20)])
@pytest.mark.parametrize("N_kv", [32, 33, 64, 65, 97, 128, 161, 290])
@pytest.mark.parametrize("at", [5, -1])
def test_edges_of_fp32_products(H, N_q, N_kv, at):
    Q, K, V = _randn(H, N_q, N_kv)
    _check(Q, K, V, _unlike("masked_key" if at > 0 else "large_value", 1e9, Q, K, V, at))


# Roundings at the size of O where nothing cancels: one a tile, of which the 75 of a wave group add up to 2^-24 sqrt(75 / 3) * 0.42 (the rms of a rounding
# over that of a number) = 1.3e-7, less what the two groups average; parts and weights make less than 1e-7 of it.  (One a product: 2.4 times as much.)
@pytest.mark.parametrize("H,N_q,N_kv", [(2, 64, 4800)])
def test_sums_of_many_tiles(H, N_q, N_kv):
    d = dev()
    Q, K, V = _randn(H, N_q, N_kv)
    Q, V = Q * 0.01, V.abs()
    O = torch.empty_like(Q, device=d)
    wk.wk_attention(Q.to(d), K.to(d), V.to(d), O)
    ref = oracle.attention(Q, K, V)
    assert np.linalg.norm(O.cpu().double().numpy() - ref) <= 1.6e-7 * np.linalg.norm(ref)


# every key at -x, whose logit has no room for anything else: even weights, whatever the size
@pytest.mark.parametrize("H,N_q,N_kv,split", [(2, 5, 1, False), (2, 64, 40, False), (300, 3, 70, False), (2, 100, 300, True)])
@pytest.mark.parametrize("x", [1e3, 1e6, 1e9, 1e10, 1e11, 1e13, 1e15])
def test_windows_far_below_0(H, N_q, N_kv, split, x):
    d = dev()
    Q, K, V = _randn(H, N_q, N_kv)
    Q[..., 0] = 1
    K[:] = 0
    K[..., 0] = -x
    n = wk.wk_attention_workspace_bytes(H, N_q, N_kv, wk.WK_F32) if split else 0
    assert (n > 0) == split
    O, lse = torch.empty_like(Q, device=d), torch.empty((H, N_q), device=d)
    wk.wk_attention(Q.to(d), K.to(d), V.to(d), O, lse, workspace=torch.empty(n, dtype=torch.uint8, device=d) if split else None)
    ref, ref_lse = oracle.attention(Q, K, V, want_lse=True)
    assert np.abs(O.cpu().double().numpy() - ref).max() <= ATT_MAX_ABS_F32
    assert np.abs(lse.cpu().double().numpy() / ref_lse - 1).max() <= 5e-7   # (parts 2^-21, a few roundings)
