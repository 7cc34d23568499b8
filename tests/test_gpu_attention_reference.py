"""bf16 attention whose scores grow behind the first tile.  The hand-scheduled loop weighs keys against the first tile's maximum and raises that
reference only when a row sum has reached 2^24; what fp32 cannot hold meanwhile is worked out again with a running maximum."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_22718_amd as wk
from wkt import K128_PAIR, K256, attention_plan, dev, frame_mask_plan

pytestmark = pytest.mark.gpu


def _levels(kind, n):
    """Of the keys, in units of 2: what is added to their scores."""
    x, at = torch.arange(n), 5 * n // 9
    return {"rises": 100.0 * x / n,                        # the reference goes up several times
            "jumps": 60.0 * (x >= at),                     # by much, inside a trip
            "falls": -100.0 * x / n,
            "beyond_fp32": 300.0 * (x >= at),
            "first_tile_without_weight": -300.0 * (x < 64),
            "values_beyond_fp32": 40.0 * (x >= at),
            "late": 110.0 * (x >= n - 290)}[kind]          # behind the last trip's first step, in the last key range alone


KINDS = ["rises", "jumps", "falls", "beyond_fp32", "first_tile_without_weight", "values_beyond_fp32", "late"]


def _inputs(kind, H, N_q, N_kv):
    g = torch.Generator().manual_seed(N_q + N_kv)
    Q, K, V = (torch.randn(H, n, 128, generator=g) for n in (N_q, N_kv, N_kv))
    Q[..., 0] = 8
    K[..., 0] = _levels(kind, N_kv) / (8 * 128 ** -0.5 * np.log2(np.e))
    if kind == "values_beyond_fp32":
        V *= 2.0 ** 100
    return [x.to(torch.bfloat16) for x in (Q, K, V)]


def _check(O, lse, rows, attend, V):
    """A weight is off by 2^-8 of itself at most (bf16, 8 significant bits), and so is the output's rounding: with A the weighted mean of |V|,
    |O - ref| <= 2^-8 (A + |ref|) + 2^-8 |ref|, and a log-sum-exp by 2^-8.  A twentieth more for scores and sums in fp32."""
    ref, ref_lse = attend(V)
    size, _ = attend(V.abs())
    got = O.float().cpu().numpy().astype(np.float64)[:, rows]
    assert np.isfinite(got).all()
    assert (np.abs(got - ref) <= 1.05 * 2.0 ** -8 * (size + 2 * np.abs(ref))).all()
    assert np.abs(lse.cpu().numpy()[:, rows] - ref_lse).max() <= 1.05 * 2.0 ** -8


def _out(Q):
    return torch.full_like(Q, float("nan"), device=dev()), torch.full(Q.shape[:2], float("nan"), device=dev())


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("H,N_q,N_kv,plan", [(2, 129, 2111, (K128_PAIR, 1)), (40, 1100, 900, (K256, 1)), (40, 1100, 600, (K256, 1)), (40, 512, 5200, (K256, 3)), (2, 300, 3000, (K128_PAIR, 8))])
def test_window(H, N_q, N_kv, plan, kind):
    d = dev()
    n = wk.wk_attention_workspace_bytes(H, N_q, N_kv, wk.WK_BF16) if plan[1] > 1 else 0
    assert attention_plan(H, N_q, N_kv, n) == plan
    Q, K, V = _inputs(kind, H, N_q, N_kv)
    O, lse = _out(Q)
    wk.wk_attention(Q.to(d), K.to(d), V.to(d), O, lse, workspace=torch.empty(n, dtype=torch.uint8, device=d) if n else None)
    rows = np.unique([r % N_q for r in (0, 31, 64, 127, 128, 200, -1)]).astype(np.int32)   # (the last 256 queries leave waves without any)
    _check(O, lse, rows, lambda v: oracle.attention(Q, K, v, rows=rows, want_lse=True), V)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("H,T,F,row0,n_after,plan", [(30, 130, 2, 320, 510, K128_PAIR), (64, 129, 3, 319, 500, K256)])
def test_frame_mask(H, T, F, row0, n_after, plan, kind):
    N_q, N_kv, d = F * T, row0 + F * T + n_after, dev()
    assert frame_mask_plan(H, N_q, N_kv, row0, T) == plan
    Q, K, V = _inputs(kind, H, N_q, N_kv)
    O, lse = _out(Q)
    ws = torch.empty(wk.wk_attention_block_causal_workspace_bytes(H, N_q), dtype=torch.uint8, device=d)
    wk.wk_attention_block_causal(Q.to(d), K.to(d), V.to(d), O, row0, T, ws, lse=lse)
    rows = np.unique([f * T + r for f in range(F) for r in (0, T // 2, T - 1)]).astype(np.int32)
    _check(O, lse, rows, lambda v: oracle.attention_block_causal(Q, K, v, row0, T, rows=rows, want_lse=True), V)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("H,layout", [(2, K128_PAIR), (100, K256)])
def test_in_place(H, layout, kind):
    N_q, n_native, n, d = 270, 64 * 14, 64 * 22 - 1, dev()
    assert attention_plan(H, N_q, n_native + n)[0] == layout and wk.lib().wk_internal_in_place_trips(n_native, 1, n)
    Q, K, V = _inputs(kind, H, N_q, n_native + n)
    store = wk.Store([K[:, n_native:].contiguous().to(d)], [V[:, n_native:].contiguous().to(d)])
    O, lse = _out(Q)
    wk.wk_attention_in_place(Q.to(d), K[:, :n_native].contiguous().to(d), V[:, :n_native].contiguous().to(d), n_native, store.desc,
                             torch.zeros(1, dtype=torch.int32, device=d), None, 1, O, lse)
    rows = np.array([0, 31, 128, 255, 256, 269], np.int32)
    _check(O, lse, rows, lambda v: oracle.attention(Q, K, v, rows=rows, want_lse=True), V)


# A run of 64 keys whose row sums lie at the end of fp32's range without leaving it: from 2^125 to 2^127 over the first tile's maximum (and at
# 2^65 and beyond the range), with nothing behind it but keys of no weight, or keys that have weight once the run is gone.
LEVELS = [60.0, 120.5, 121.0, 121.5, 122.0, 122.5, 124.5]


def _run_inputs(level, behind, H, N_q, N_kv, at):
    g = torch.Generator().manual_seed(N_q + N_kv)
    Q, K, V = (torch.randn(H, n, 128, generator=g) for n in (N_q, N_kv, N_kv))
    K *= 0.1   # (a run's sums are 2^5 of its level, row for row)
    Q[..., 0] = 8
    K[..., 0] = 0
    K[:, at + 64:, 0] = 100.0 if behind else 0.0
    K[:, at:at + 64, 0] = level
    K[..., 0] /= 8 * 128 ** -0.5 * np.log2(np.e)
    return [x.to(torch.bfloat16) for x in (Q, K, V * 2.0 ** -10)]   # (outputs stay within fp32 while they are summed)


@pytest.mark.parametrize("behind", [False, True])
@pytest.mark.parametrize("level", LEVELS)
@pytest.mark.parametrize("H,N_q,N_kv,plan", [(2, 129, 2111, (K128_PAIR, 1)), (40, 1100, 900, (K256, 1)), (40, 1100, 2100, (K256, 1)), (40, 512, 5200, (K256, 3)),
                                             (2, 300, 3000, (K128_PAIR, 8))])
def test_sums_at_the_end_of_the_range(H, N_q, N_kv, plan, level, behind):
    d = dev()
    n = wk.wk_attention_workspace_bytes(H, N_q, N_kv, wk.WK_BF16) if plan[1] > 1 else 0
    assert attention_plan(H, N_q, N_kv, n) == plan
    Q, K, V = _run_inputs(level, behind, H, N_q, N_kv, 5 * N_kv // 9 // 64 * 64)
    O, lse = _out(Q)
    wk.wk_attention(Q.to(d), K.to(d), V.to(d), O, lse, workspace=torch.empty(n, dtype=torch.uint8, device=d) if n else None)
    rows = np.unique([r % N_q for r in (0, 31, 64, 127, 128, 200, -1)]).astype(np.int32)
    _check(O, lse, rows, lambda v: oracle.attention(Q, K, v, rows=rows, want_lse=True), V)


@pytest.mark.parametrize("behind", [False, True])
@pytest.mark.parametrize("level", LEVELS)
@pytest.mark.parametrize("H,T,F,row0,n_after,plan", [(30, 130, 2, 320, 510, K128_PAIR), (64, 129, 3, 319, 500, K256)])
def test_sums_at_the_end_of_the_range_frame_mask(H, T, F, row0, n_after, plan, level, behind):
    N_q, N_kv, d = F * T, row0 + F * T + n_after, dev()
    assert frame_mask_plan(H, N_q, N_kv, row0, T) == plan
    Q, K, V = _run_inputs(level, behind, H, N_q, N_kv, row0 + F * T)
    O, lse = _out(Q)
    ws = torch.empty(wk.wk_attention_block_causal_workspace_bytes(H, N_q), dtype=torch.uint8, device=d)
    wk.wk_attention_block_causal(Q.to(d), K.to(d), V.to(d), O, row0, T, ws, lse=lse)
    rows = np.unique([f * T + r for f in range(F) for r in (0, T // 2, T - 1)]).astype(np.int32)
    _check(O, lse, rows, lambda v: oracle.attention_block_causal(Q, K, v, row0, T, rows=rows, want_lse=True), V)


@pytest.mark.parametrize("behind", [False, True])
@pytest.mark.parametrize("level", LEVELS)
@pytest.mark.parametrize("H,layout", [(2, K128_PAIR), (100, K256)])
@pytest.mark.parametrize("at", [64 * 6, 64 * 19])   # in either segment
def test_sums_at_the_end_of_the_range_in_place(at, H, layout, level, behind):
    N_q, n_native, n, d = 270, 64 * 14, 64 * 22 - 1, dev()
    assert attention_plan(H, N_q, n_native + n)[0] == layout and wk.lib().wk_internal_in_place_trips(n_native, 1, n)
    Q, K, V = _run_inputs(level, behind, H, N_q, n_native + n, at)
    store = wk.Store([K[:, n_native:].contiguous().to(d)], [V[:, n_native:].contiguous().to(d)])
    O, lse = _out(Q)
    wk.wk_attention_in_place(Q.to(d), K[:, :n_native].contiguous().to(d), V[:, :n_native].contiguous().to(d), n_native, store.desc,
                             torch.zeros(1, dtype=torch.int32, device=d), None, 1, O, lse)
    rows = np.array([0, 31, 128, 255, 256, 269], np.int32)
    _check(O, lse, rows, lambda v: oracle.attention(Q, K, v, rows=rows, want_lse=True), V)


# Waves of a workgroup part where only some of its queries see the growth: their results are in place when the others' work is done once more.
@pytest.mark.parametrize("alias", [False, True])   # (the second pass of a wave whose results are in place has lost its queries where they take their place)
@pytest.mark.parametrize("H,N_q,N_kv,plan", [(40, 1100, 900, (K256, 1)), (40, 512, 5200, (K256, 3)), (2, 300, 3000, (K128_PAIR, 1))])
def test_growth_for_some_waves(H, N_q, N_kv, plan, alias):
    d = dev()
    n = wk.wk_attention_workspace_bytes(H, N_q, N_kv, wk.WK_BF16) if plan[1] > 1 else 0
    assert attention_plan(H, N_q, N_kv, n) == plan
    Q, K, V = _inputs("beyond_fp32", H, N_q, N_kv)
    q = torch.arange(N_q)
    Q[:, (q < 32) | (q >= 64) & (q < 224), 0] = 0   # of the first workgroup of 256 one wave and a wave's neighbour see it, of the others all
    O, lse = _out(Q)
    queries = Q.to(d)
    if alias and plan[1] == 1:
        O = queries
    wk.wk_attention(queries, K.to(d), V.to(d), O, lse, workspace=torch.empty(n, dtype=torch.uint8, device=d) if n else None)
    rows = np.unique([0, 31, 32, 63, 64, 100, 223, 224, 255, 256, N_q - 1]).astype(np.int32)
    _check(O, lse, rows, lambda v: oracle.attention(Q, K, v, rows=rows, want_lse=True), V)
