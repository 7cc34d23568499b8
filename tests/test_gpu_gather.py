"""GPU parity of wk_gather_window against the oracle: byte-exact window assembly (Sec. 4.2)."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2605_22718_amd as wk
import wk_synth as ws
from wkt import bits, dev

pytestmark = pytest.mark.gpu


def _store(cfg, lengths, pinned=False):
    ks, vs = [], []
    for c, n in enumerate(lengths):
        k, v = ws.make_native(cfg.with_(index=50 + c), n_rows=n)
        ks.append(k), vs.append(v)
    if pinned:
        place = lambda t: t.clone().pin_memory()
    else:
        place = lambda t: t.to(dev())
    return ks, vs, wk.Store([place(k) for k in ks], [place(v) for v in vs])


def _gather(cfg, store, ids, n_ids, R_max, Kn, Vn, cap, in_place=False):
    d = dev()
    Kw = torch.full((cfg.H, cap, cfg.d), 7.0, dtype=ws.torch_dtype(cfg.dtype), device=d)
    Vw = torch.full_like(Kw, 9.0)
    n_native = Kn.shape[1]
    if in_place:
        Kw[:, :n_native] = Kn.to(d)
        Vw[:, :n_native] = Vn.to(d)
    n_win = torch.full((1,), -1, dtype=torch.int32, device=d)
    ids_d = torch.tensor(list(ids) + [0] * (R_max - len(ids)), dtype=torch.int32, device=d) if R_max else None
    n_ids_d = None if n_ids is None else torch.tensor([n_ids], dtype=torch.int32, device=d)
    wk.wk_gather_window(store.desc, ids_d, n_ids_d, R_max, None if in_place else Kn.to(d),
                        None if in_place else Vn.to(d), n_native, Kw, Vw, cap, n_win)
    torch.cuda.synchronize()
    return Kw.cpu(), Vw.cpu(), int(n_win.item())


@pytest.mark.parametrize("dtype", [ws.configs.DT_BF16, ws.configs.DT_F32])
@pytest.mark.parametrize("pinned", [False, True])
def test_gather_matches_oracle(dtype, pinned):
    cfg = ws.get_config(1).with_(H=3, dtype=dtype)
    lengths = [5, 300, 77, 1, 129, 64]
    ks, vs, store = _store(cfg, lengths, pinned)
    Kn, Vn = ws.make_native(cfg, n_rows=131)
    cap = 131 + 4 * 300
    for ids in ([1, 0, 5, 2], [3], [], [4, 4, 1]):
        Kw, Vw, n_win = _gather(cfg, store, ids, len(ids), 4, Kn, Vn, cap)
        oK, oV, o_n = oracle.gather(ks, vs, ids, Kn, Vn, cap)
        assert n_win == o_n
        assert torch.equal(bits(Kw[:, :n_win]), bits(oK[:, :n_win])) and torch.equal(bits(Vw[:, :n_win]), bits(oV[:, :n_win]))
        assert (Kw[:, n_win:] == 7).all() and (Vw[:, n_win:] == 9).all()     # rows past the window untouched
    # n_ids = NULL uses all R_max ids; invalid ids are skipped
    Kw, Vw, n_win = _gather(cfg, store, [2, -1, 99, 0], None, 4, Kn, Vn, cap)
    oK, oV, o_n = oracle.gather(ks, vs, [2, 0], Kn, Vn, cap)
    assert n_win == o_n and torch.equal(bits(Kw[:, :n_win]), bits(oK[:, :n_win]))
    # native rows already in place
    Kw, Vw, n_win = _gather(cfg, store, [5, 1], 2, 4, Kn, Vn, cap, in_place=True)
    oK, oV, o_n = oracle.gather(ks, vs, [5, 1], Kn, Vn, cap)
    assert n_win == o_n and torch.equal(bits(Kw[:, :n_win]), bits(oK[:, :n_win])) and torch.equal(bits(Vw[:, :n_win]), bits(oV[:, :n_win]))


def test_no_native_rows_and_no_retrieval():
    cfg = ws.get_config(1).with_(H=2)
    ks, vs, store = _store(cfg, [40, 40])
    empty = torch.zeros((2, 0, 128), dtype=torch.bfloat16)
    Kw, Vw, n_win = _gather(cfg, store, [1, 0], 2, 2, empty, empty, 80)
    oK, oV, o_n = oracle.gather(ks, vs, [1, 0], None, None, 80)
    assert n_win == 80 and torch.equal(bits(Kw), bits(oK)) and torch.equal(bits(Vw), bits(oV))
    Kn, Vn = ws.make_native(cfg, n_rows=33)
    Kw, Vw, n_win = _gather(cfg, store, [], 0, 0, Kn, Vn, 33)     # R_max = 0: sliding window only
    assert n_win == 33 and torch.equal(bits(Kw), bits(Kn)) and torch.equal(bits(Vw), bits(Vn))


@pytest.mark.parametrize("ci,order", [(1, (4, 0, 5, 2)), (2, (9, 4, 0, 5, 2, 11, 7, 1))])
def test_config_sized_gather(ci, order):
    """Configs 1 and 2 at full size from an HBM store, in the launch the bench times (ids on the device)."""
    cfg = ws.get_config(ci)
    d = dev()
    n_out, _ = wk.wk_keep_count(cfg.rho, cfg.ratio_kind, cfg.anchor_mode, cfg.F, cfg.T)
    ks = [ws.make_native(cfg.with_(index=70 + c), d, n_rows=n_out) for c in range(12)]
    store = wk.Store([k for k, _ in ks], [v for _, v in ks])
    Kn, Vn = ws.make_native(cfg, d)
    cap = cfg.n_native + cfg.R * n_out
    Kw = torch.zeros((cfg.H, cap, cfg.d), dtype=torch.bfloat16, device=d)
    Vw = torch.zeros_like(Kw)
    ids = torch.tensor(order, dtype=torch.int32, device=d)
    n_win = torch.zeros(1, dtype=torch.int32, device=d)
    wk.wk_gather_window(store.desc, ids, None, cfg.R, Kn, Vn, cfg.n_native, Kw, Vw, cap, n_win)
    torch.cuda.synchronize()
    assert int(n_win.item()) == cap == (10560 if ci == 1 else 28080)
    expect_k = torch.cat([Kn] + [ks[i][0] for i in order], 1)
    expect_v = torch.cat([Vn] + [ks[i][1] for i in order], 1)
    assert torch.equal(bits(Kw), bits(expect_k)) and torch.equal(bits(Vw), bits(expect_v))
    # byte-exact against the oracle on one head's slice (the oracle copies on the CPU)
    oK, oV, _ = oracle.gather([k[:1].cpu() for k, _ in ks], [v[:1].cpu() for _, v in ks], list(order),
                              Kn[:1].cpu(), Vn[:1].cpu(), cap)
    assert torch.equal(bits(Kw[:1].cpu()), bits(oK)) and torch.equal(bits(Vw[:1].cpu()), bits(oV))
    # native rows already in place: only the retrieved chunks move, same window
    Kw2, Vw2 = torch.zeros_like(Kw), torch.zeros_like(Vw)
    Kw2[:, :cfg.n_native], Vw2[:, :cfg.n_native] = Kn, Vn
    wk.wk_gather_window(store.desc, ids, None, cfg.R, None, None, cfg.n_native, Kw2, Vw2, cap, n_win)
    torch.cuda.synchronize()
    assert torch.equal(bits(Kw2), bits(expect_k)) and torch.equal(bits(Vw2), bits(expect_v))


def test_calibration_copy_is_exact():
    d = dev()
    g = torch.Generator(device="cpu").manual_seed(1)
    for n in (16, 48, 32 * 1024 + 16, 5 * 1024 * 1024 + 32):
        src = torch.randint(0, 255, (n,), dtype=torch.uint8, generator=g).to(d)
        dst = torch.zeros(n + 16, dtype=torch.uint8, device=d)
        wk.wk_calibration_copy(dst[:n], src)
        torch.cuda.synchronize()
        assert torch.equal(dst[:n], src) and int(dst[n:].sum()) == 0


def test_chunks_beyond_the_descriptors_bound_are_skipped():
    """max_tok is a hard bound: a chunk whose n_tok exceeds it is skipped (its head stride is its true length,
    so it cannot be read cut short), by the gather and by attention in place alike."""
    import ctypes as C
    cfg = ws.get_config(1).with_(H=3)
    lengths = [40, 300, 77, 129]
    ks, vs, store = _store(cfg, lengths)
    tight = wk.wk_store_desc(store.K_ptr.data_ptr(), store.V_ptr.data_ptr(), store.n_tok.data_ptr(), len(lengths),
                             129, cfg.H, cfg.d, store.dtype)          # chunk 1 (300 rows) violates the bound
    Kn, Vn = ws.make_native(cfg, n_rows=70)
    ids = [3, 1, 0, 2]
    cap = 70 + 4 * 129
    d = dev()
    Kw = torch.full((cfg.H, cap, cfg.d), 7.0, dtype=torch.bfloat16, device=d)
    Vw = torch.full_like(Kw, 9.0)
    n_win = torch.full((1,), -1, dtype=torch.int32, device=d)
    ids_d = torch.tensor(ids, dtype=torch.int32, device=d)
    wk.wk_gather_window(tight, ids_d, None, 4, Kn.to(d), Vn.to(d), 70, Kw, Vw, cap, n_win)
    torch.cuda.synchronize()
    oK, oV, o_n = oracle.gather(ks, vs, [3, 0, 2], Kn, Vn, cap)
    assert int(n_win.item()) == o_n == 70 + 129 + 40 + 77
    assert torch.equal(bits(Kw.cpu()[:, :o_n]), bits(oK[:, :o_n])) and torch.equal(bits(Vw.cpu()[:, :o_n]), bits(oV[:, :o_n]))
    assert (Kw[:, o_n:] == 7).all()
    # attention in place skips the same chunk
    Q = ws.make_queries(cfg, n_q=90)
    O = torch.empty((cfg.H, 90, cfg.d), dtype=torch.bfloat16, device=d)
    lse = torch.empty((cfg.H, 90), dtype=torch.float32, device=d)
    wk.wk_attention_in_place(Q.to(d), Kn.to(d), Vn.to(d), 70, tight, ids_d, None, 4, O, lse)
    torch.cuda.synchronize()
    ref, ref_lse = oracle.attention(Q, oK, oV, N_kv=o_n, want_lse=True)
    err = np.abs(O.float().cpu().numpy().astype(np.float64) - ref)
    assert err.max() <= 2e-2 and err.mean() <= 2e-3
    assert np.abs(lse.cpu().numpy() - ref_lse).max() <= 2e-2
    # the chunk index for query-based retrieval reports such a chunk as empty
    out = torch.empty((len(lengths), cfg.H, 90), dtype=torch.float32, device=d)
    wk.wk_chunk_lse(tight, Q.to(d), out)
    torch.cuda.synchronize()
    assert torch.isinf(out[1]).all() and (out[1] < 0).all() and torch.isfinite(out[[0, 2, 3]]).all()


def test_id_list_no_longer_than_its_count():
    """Only the first *n_ids ids are read: here the list ends with them, R_max is larger."""
    cfg = ws.get_config(1).with_(H=2)
    ks, vs, store = _store(cfg, [40, 70, 20])
    d = dev()
    Kw, Vw = (torch.zeros((2, 4 * 70, 128), dtype=torch.bfloat16, device=d) for _ in range(2))
    n_win = torch.empty(1, dtype=torch.int32, device=d)
    wk.wk_gather_window(store.desc, torch.tensor([2, 1], dtype=torch.int32, device=d), torch.tensor([2], dtype=torch.int32, device=d), 4,
                        None, None, 0, Kw, Vw, 4 * 70, n_win)
    assert int(n_win.item()) == 90 and torch.equal(bits(Kw[:, :90].cpu()), bits(torch.cat([ks[2], ks[1]], 1)))


def test_more_units_than_a_launch_has_workgroups_of_512():
    """A row each of 2^22 + 1 heads: 2^23 + 2 work units, where 2^23 workgroups of 512 threads are a launch's limit."""
    d, H = dev(), 2 ** 22 + 1
    g = torch.Generator(device=d).manual_seed(1)
    K, V = [torch.randint(-2 ** 61, 2 ** 61, (H, 1, 32), generator=g, device=d).view(torch.bfloat16) for _ in range(2)]
    store = wk.Store([K], [V])
    Kw, Vw = [torch.zeros((H, 1, 128), dtype=torch.bfloat16, device=d) for _ in range(2)]
    n_win = torch.empty(1, dtype=torch.int32, device=d)
    wk.wk_gather_window(store.desc, torch.zeros(1, dtype=torch.int32, device=d), None, 1, None, None, 0, Kw, Vw, 1, n_win)
    assert int(n_win) == 1
    assert torch.equal(bits(Kw), bits(K)) and torch.equal(bits(Vw), bits(V))


# the segments in a wave's lanes (up to 63 chunks) and in LDS: counts at either side of that, chunks of a few rows, so that a work unit lies
# across dozens of them, empty ones, ids outside the store, native rows in place, copied and none
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("R,n_ids,n_native,native", [(0, 0, 70, True), (1, 1, 0, False), (62, 62, 5, True), (63, 63, 0, False), (63, 40, 129, False),
                                                     (64, 64, 5, True), (65, 65, 33, False), (63, 63, 700, True)])
def test_segments_in_lanes_and_in_lds(R, n_ids, n_native, native, dtype):
    H, M, d = 3, 70, dev()
    g = torch.Generator().manual_seed(R + n_native)
    lens = [(11 * i) % 9 * (40 if i % 13 == 0 else 1) for i in range(M)]   # 0 to 320 rows
    ks, vs = ([torch.randn((H, n, 128), generator=g).to(dtype).to(d) for n in lens] for _ in range(2))
    store = wk.Store(ks, vs)
    ids = torch.randperm(M, generator=g)[:max(R, 1)].to(torch.int32)
    if R > 4:
        ids[3], ids[4] = -1, M
    cap = n_native + R * store.max_tok
    Kn, Vn = (torch.randn((H, n_native, 128), generator=g).to(dtype).to(d) for _ in range(2))
    Kw, Vw = (torch.full((H, max(cap, 1), 128), 7.0, dtype=dtype, device=d) for _ in range(2))
    want = []
    for w, nat, chunks in ((Kw, Kn, ks), (Vw, Vn, vs)):
        rows = torch.cat([nat if native else w[:, :n_native].clone()] + [chunks[i] for i in ids[:n_ids].tolist() if 0 <= i < M], 1)
        want.append(torch.cat([rows, w[:, rows.shape[1]:]], 1))
        n = rows.shape[1]
    n_win = torch.zeros(1, dtype=torch.int32, device=d)
    wk.wk_gather_window(store.desc, ids.to(d), torch.tensor([n_ids], dtype=torch.int32, device=d), R, Kn if native else None, Vn if native else None,
                        n_native, Kw, Vw, cap, n_win)
    assert n_win.item() == n and torch.equal(Kw, want[0]) and torch.equal(Vw, want[1])


# copies of few work units are made in smaller ones: heads of one unit of 96 rows, either side of the two bounds, and 24 KB in 256 threads behind them
@pytest.mark.parametrize("H,pieces", [(1, 3), (12, 3), (13, 2), (180, 2), (181, 1)])
@pytest.mark.parametrize("native", [True, False])
@pytest.mark.parametrize("pinned", [True, False])   # (the first load tells)
def test_smaller_units_for_few(H, pieces, native, pinned):
    f = wk.lib().wk_internal_gather_threads
    f.argtypes, f.restype = [ctypes.c_int32, ctypes.c_int64, ctypes.c_int32, ctypes.c_int32], ctypes.c_int64
    assert f(H, 96, wk.WK_BF16, 0) == 2 * H * pieces * 256
    n_native, lens, d = 7, [44 if native else 48, 37, 5], dev()   # 95 or 96 rows to copy at most: one unit of 24 KB
    g = torch.Generator().manual_seed(H)
    ks, vs = ([torch.randn((H, n, 128), generator=g).to(torch.bfloat16).to(d) for n in lens] for _ in range(2))
    store = wk.Store(*([x.cpu().pin_memory() for x in c] for c in (ks, vs))) if pinned else wk.Store(ks, vs)
    Kn, Vn = (torch.randn((H, n_native, 128), generator=g).to(torch.bfloat16).to(d) for _ in range(2))
    cap = n_native + 2 * store.max_tok
    Kw, Vw = (torch.full((H, cap, 128), 7.0, dtype=torch.bfloat16, device=d) for _ in range(2))
    n_win = torch.zeros(1, dtype=torch.int32, device=d)
    wk.wk_gather_window(store.desc, torch.tensor([1, 0], dtype=torch.int32, device=d), None, 2, Kn if native else None, Vn if native else None,
                        n_native, Kw, Vw, cap, n_win)
    n = n_native + lens[1] + lens[0]
    assert n_win.item() == n
    for w, nat, chunks in ((Kw, Kn, ks), (Vw, Vn, vs)):
        assert torch.equal(w[:, :n_native], nat if native else torch.full_like(nat, 7.0))
        assert torch.equal(w[:, n_native:n], torch.cat([chunks[1], chunks[0]], 1)) and (w[:, n:] == 7.0).all()
