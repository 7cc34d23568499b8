"""The work that users of the WorldKV hot path have it do, as cases that can be timed and compared.

Every case is one pass through the public entry points of `paper_2605_22718_amd`, called as a rollout calls them:
buffers, stores, descriptors and workspaces are made once, inputs are resident where the path expects them, nothing
synchronises.  Sizes are those of the repository's five workloads (880 and 1,560 tokens per latent frame, 12 and 40
heads, head dimension 128, chunks of three frames) and ragged sizes of the same ranges.

The kinds:

  poses     top-R retrieval by camera pose over the whole store (once per denoising step)
  step      one layer of one denoising step: compress the evicted chunk, retrieve, assemble the window, attend
  attention softmax attention over a window that is already assembled
  compress  World Compression of one chunk or of a batch (eviction; building a store from a recorded rollout)
  query     query-based retrieval: log-sum-exp of the queries against every stored chunk, then the top-R masses
  in_place  attention over native rows and retrieved chunks where an HBM-resident store keeps them
  causal    attention with the frame-level mask inside the chunk being denoised
  refresh   two consecutive denoising steps of a smooth camera path over a store in pinned host memory: one of
            the R retrieved chunks changes per step and is fetched over the host link, then attention
"""
import math

import torch

import paper_2605_22718_amd as wk
import wk_synth as ws

D = 128
_DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
_KINDS = ("poses", "step", "attention", "compress", "query", "in_place", "causal", "refresh")


def listed():
    return [
        # retrieval over a long rollout's store (1,000 chunks, budget 16): the smallest call, launch latency and one workgroup's work
        dict(name="poses_1000", kind="poses", M=1000, R=16),
        # the tiny workload: 4 heads, one 880-token frame, fp32, one-frame chunks with an external anchor
        dict(name="tiny_step_f32", kind="step", dtype="f32", H=4, T=880, F=1, external=True, q_frames=1, native_frames=2,
             M=16, R=2, rho=0.5),
        # one layer and step of the Matrix-Game-2.0-shaped rollout (12 heads, 880 tokens per frame)
        dict(name="matrix_game_step", kind="step", dtype="bf16", H=12, T=880, F=3, external=False, q_frames=3,
             native_frames=6, M=60, R=4, rho=0.5),
        # one layer and step of the LingBot-World-Fast-shaped rollout (40 heads, 1,560 tokens per frame), store in HBM
        dict(name="lingbot_step", kind="step", dtype="bf16", H=40, T=1560, F=3, external=False, q_frames=3,
             native_frames=6, M=120, R=8, rho=0.5),
        # the baseline the method avoids: every key of a one-minute rollout
        dict(name="full_kv_attention", kind="attention", dtype="bf16", H=12, N_q=2640, N_kv=211200, pad=0, lse=False),
        # a store built from a recorded rollout: 64 chunks in one call, half of the non-anchor tokens kept
        dict(name="compress_batch64", kind="compress", dtype="bf16", H=40, T=1560, F=3, batch=64, rho=0.5,
             ratio="nonanchor", heads="shared", algo="factored"),
        # one evicted chunk with an index set per head, ragged sizes
        dict(name="compress_per_head", kind="compress", dtype="bf16", H=24, T=1013, F=3, batch=1, rho=0.5, ratio="chunk",
             heads="independent", algo="factored"),
        # the similarity product on the matrix cores, one evicted chunk per layer of a 4-layer group
        dict(name="compress_gemm", kind="compress", dtype="bf16", H=40, T=1560, F=3, batch=4, rho=0.25, ratio="nonanchor",
             heads="shared", algo="gemm"),
        # query-based retrieval over the anchor keys of 120 stored chunks
        dict(name="query_lingbot", kind="query", dtype="bf16", H=40, N_q=4680, M=120, tokens=1560, R=8),
        # a ragged window read in place: 16 heads, chunks of different lengths, a native part that fills no whole tile
        dict(name="in_place_ragged", kind="in_place", dtype="bf16", H=16, N_q=3333, n_native=6101, M=24, R=7, tokens=1747),
        # frame-causal attention, Matrix-Game shape: sink chunk, the chunk being denoised, retrieved chunks behind it
        dict(name="causal_matrix_game", kind="causal", dtype="bf16", H=12, T=880, q_frames=3, N_kv=10560, row0=2640),
        # the offloaded store of a smooth camera path (one changed chunk per step), Matrix-Game shape
        dict(name="refresh_matrix_game", kind="refresh", dtype="bf16", H=12, T=880, q_frames=3, native_frames=6, M=24, R=4,
             tokens=1320),
    ]


# ---- drawn cases: the same kinds over their ranges ------------------------------------------------------------

def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_kind(rng, kind):
    f32 = rng.random() < 0.25
    dtype = "f32" if f32 else "bf16"
    H, T = _log_int(rng, 2, 40), _log_int(rng, 64, 1560)
    if kind == "poses":
        return dict(kind=kind, M=_log_int(rng, 4, 4096), R=_log_int(rng, 1, 32))
    if kind == "step":
        external = rng.random() < 0.2
        M = rng.randint(4, 48)
        return dict(kind=kind, dtype=dtype, H=H, T=T, F=1 if external else 3, external=external, q_frames=rng.randint(1, 3),
                    native_frames=rng.randint(3, 6), M=M, R=rng.randint(1, min(M, 9)), rho=rng.choice((0.4, 0.5, 0.75)))
    if kind == "attention":
        return dict(kind=kind, dtype=dtype, H=H, N_q=_log_int(rng, 64, 4680), N_kv=_log_int(rng, 256, 211200),
                    pad=rng.choice((0, 0, rng.randint(1, 999))), lse=rng.random() < 0.5)
    if kind == "compress":
        heads = rng.choice(("shared", "shared", "independent"))
        algo = "gemm" if not f32 and rng.random() < 0.25 else "factored"
        return dict(kind=kind, dtype=dtype, H=H, T=T, F=3, batch=_log_int(rng, 1, 64), rho=rng.choice((0.25, 0.5, 0.75)),
                    ratio="nonanchor", heads=heads, algo=algo)
    if kind == "query":
        M = _log_int(rng, 4, 400)
        return dict(kind=kind, dtype="bf16", H=H, N_q=_log_int(rng, 128, 4680), M=M, tokens=T, R=rng.randint(1, min(M, 16)))
    if kind == "in_place":
        R = rng.randint(1, 16)
        return dict(kind=kind, dtype="bf16", H=H, N_q=_log_int(rng, 128, 4680), n_native=_log_int(rng, 256, 9360),
                    M=R + rng.randint(0, 8), R=R, tokens=_log_int(rng, 96, 2340))
    if kind == "causal":
        q_frames = rng.randint(1, 3)
        row0 = rng.randint(0, 2) * T
        return dict(kind=kind, dtype=dtype, H=H, T=T, q_frames=q_frames, N_kv=row0 + q_frames * T + rng.randint(0, 12) * T // 2,
                    row0=row0)
    R = rng.randint(1, 6)
    return dict(kind="refresh", dtype="bf16", H=_log_int(rng, 2, 16), T=T, q_frames=rng.randint(1, 3), native_frames=rng.randint(3, 6),
                M=R + rng.randint(1, 12), R=R, tokens=T + rng.randint(0, T))


def draw(rng):
    """One more case: a kind, then sizes over that kind's range until the pass costs no more than the listed ones."""
    kind = rng.choice(_KINDS)
    while True:
        c = _draw_kind(rng, kind)
        w = work(c)
        # fp32 products run on matrix instructions of a sixteenth of the bf16 rate
        if w["bytes"] <= 1e10 and w["flops"] <= (1.5e11 if c.get("dtype") == "f32" else 3.4e12):
            return c


# ---- inputs ------------------------------------------------------------------------------------------------------

def _randn(gen, shape, dtype):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).to(dtype)


def _chunk(gen, H, T, F, external, dtype):
    """One evicted chunk's K and V [H][F*T][d] (and external anchor): a non-anchor token is, with probability one half,
    the anchor token at its place plus noise (one choice per token for all heads, K and V), else fresh."""
    first = 0 if external else 1
    anchor_k, anchor_v = _randn(gen, (H, T, D), torch.float32), _randn(gen, (H, T, D), torch.float32)
    k, v = ([], []) if external else ([anchor_k], [anchor_v])
    for _ in range(first, F):
        copy = (torch.rand(T, generator=gen, device="cuda") < 0.5).view(1, T, 1)
        for out, anchor in ((k, anchor_k), (v, anchor_v)):
            fresh = _randn(gen, (H, T, D), torch.float32)
            out.append(torch.where(copy, anchor + 0.05 * fresh, fresh))
    return torch.cat(k, 1).to(dtype), torch.cat(v, 1).to(dtype), anchor_k.to(dtype) if external else None


def _bytes(n):
    return torch.empty(n, dtype=torch.uint8, device="cuda") if n else None


def _int32(n):
    return torch.zeros(n, dtype=torch.int32, device="cuda")


def _ids(gen, M, R):
    return torch.randperm(M, generator=gen, device="cuda")[:R].to(torch.int32)


def _attention_workspace(H, N_q, N_kv, dtype):
    return _bytes(wk.wk_attention_workspace_bytes(H, N_q, N_kv, wk.WK_BF16 if dtype == torch.bfloat16 else wk.WK_F32))


def _compress_desc(c, batch=1):
    return wk.make_compress_desc(
        c["H"], c["T"], c["F"], wk.WK_BF16 if c["dtype"] == "bf16" else wk.WK_F32, c["rho"], batch=batch,
        head_mode=wk.WK_HEADS_INDEPENDENT if c.get("heads") == "independent" else wk.WK_HEADS_SHARED,
        anchor_mode=wk.WK_ANCHOR_EXTERNAL if c.get("external") else wk.WK_ANCHOR_FIRST_FRAME,
        ratio_kind=wk.WK_RATIO_NONANCHOR if c.get("ratio") == "nonanchor" else wk.WK_RATIO_CHUNK,
        score_algo=wk.WK_SCORE_GEMM if c.get("algo") == "gemm" else wk.WK_SCORE_FACTORED)


def _poses(M, seed):
    poses, cur = ws.make_poses(M, seed)   # looping trajectory that comes back to where it began
    return torch.from_numpy(poses).cuda(), [float(x) for x in cur]


def prepare(case, seed):
    c, gen = case, torch.Generator(device="cuda").manual_seed(seed)
    return {"case": c, **globals()["_prepare_" + c["kind"]](c, gen, seed)}


def _prepare_poses(c, gen, seed):
    poses, cur = _poses(c["M"], seed)
    return dict(poses=poses, cur=cur, ids=_int32(c["R"]), n_found=_int32(1),
                dist=torch.zeros(c["R"], dtype=torch.float64, device="cuda"))


def _prepare_step(c, gen, seed):
    H, T, M, R, dt = c["H"], c["T"], c["M"], c["R"], _DTYPES[c["dtype"]]
    desc = _compress_desc(c)
    n_out, _ = wk.wk_keep_count(desc.rho, desc.ratio_kind, desc.anchor_mode, c["F"], T)
    n_native, N_q = c["native_frames"] * T, c["q_frames"] * T
    cap = n_native + R * n_out
    K, V, A = _chunk(gen, H, T, c["F"], c["external"], dt)
    store_k, store_v = ([_randn(gen, (H, n_out, D), dt) for _ in range(M)] for _ in range(2))
    K_win, V_win = _randn(gen, (H, cap, D), dt), _randn(gen, (H, cap, D), dt)   # rows [0, n_native) are the native ones
    s = _prepare_poses(c, gen, seed)
    return dict(s, desc=desc, K=K, V=V, A=A, kept=_int32((1, n_out)), K_out=torch.empty((H, n_out, D), dtype=dt, device="cuda"),
                V_out=torch.empty((H, n_out, D), dtype=dt, device="cuda"), ws=_bytes(wk.wk_compress_workspace_bytes(desc)),
                store=wk.Store(store_k, store_v), n_native=n_native, cap=cap, K_win=K_win, V_win=V_win, n_win=_int32(1),
                Q=_randn(gen, (H, N_q, D), dt), O=torch.empty((H, N_q, D), dtype=dt, device="cuda"),
                att_ws=_attention_workspace(H, N_q, cap, dt))


def _prepare_attention(c, gen, seed):
    H, N_q, N_kv, dt = c["H"], c["N_q"], c["N_kv"], _DTYPES[c["dtype"]]
    return dict(Q=_randn(gen, (H, N_q, D), dt), K_win=_randn(gen, (H, N_kv + c["pad"], D), dt),
                V_win=_randn(gen, (H, N_kv + c["pad"], D), dt), O=torch.empty((H, N_q, D), dtype=dt, device="cuda"),
                lse=torch.empty((H, N_q), device="cuda") if c["lse"] else None, att_ws=_attention_workspace(H, N_q, N_kv, dt))


def _prepare_compress(c, gen, seed):
    H, T, F, B, dt = c["H"], c["T"], c["F"], c["batch"], _DTYPES[c["dtype"]]
    desc = _compress_desc(c, B)
    n_out, _ = wk.wk_keep_count(desc.rho, desc.ratio_kind, desc.anchor_mode, F, T)
    K, V = torch.empty((B, H, F * T, D), dtype=dt, device="cuda"), torch.empty((B, H, F * T, D), dtype=dt, device="cuda")
    for b in range(B):
        K[b], V[b], _ = _chunk(gen, H, T, F, False, dt)
    G = H if c["heads"] == "independent" else 1
    ws_bytes = _bytes(wk.wk_compress_workspace_bytes(desc))
    scores = ws_bytes[:B * G * (F - 1) * T * 8].view(torch.float64)   # where the call leaves the redundancy scores
    return dict(desc=desc, K=K, V=V, kept=_int32((B, G, n_out)), K_out=torch.empty((B, H, n_out, D), dtype=dt, device="cuda"),
                V_out=torch.empty((B, H, n_out, D), dtype=dt, device="cuda"), ws=ws_bytes, scores=scores)


def _prepare_query(c, gen, seed):
    H, N_q, M, n, dt = c["H"], c["N_q"], c["M"], c["tokens"], _DTYPES[c["dtype"]]
    Q = _randn(gen, (H, N_q, D), dt)
    # a chunk that shows what the queries look at has keys aligned with them, more or less by chunk
    a = torch.rand(M, generator=gen, device="cuda") * 0.6
    keys = []
    for i in range(M):
        rows = (7 * torch.arange(n, device="cuda") + i) % N_q
        keys.append((_randn(gen, (H, n, D), torch.float32) + a[i] * Q[:, rows]).to(dt))
    return dict(Q=Q, store=wk.Store(keys, keys), lse=torch.empty((M, H, N_q), device="cuda"), ids=_int32(c["R"]), n_found=_int32(1),
                mass=torch.zeros(c["R"], dtype=torch.float64, device="cuda"),
                ws=_bytes(wk.wk_score_chunks_query_workspace_bytes(M, H * N_q)))


def _chunk_lengths(c):
    """Stored lengths that differ from chunk to chunk, as ratios that differ along a rollout leave them."""
    return [max(1, c["tokens"] - (37 * i) % (1 + c["tokens"] // 3)) for i in range(c["M"])]


def _prepare_in_place(c, gen, seed):
    H, N_q, dt = c["H"], c["N_q"], _DTYPES[c["dtype"]]
    keys, values = ([_randn(gen, (H, n, D), dt) for n in _chunk_lengths(c)] for _ in range(2))
    return dict(Q=_randn(gen, (H, N_q, D), dt), K_nat=_randn(gen, (H, c["n_native"], D), dt), V_nat=_randn(gen, (H, c["n_native"], D), dt),
                store=wk.Store(keys, values), ids=torch.arange(c["R"], device="cuda").to(torch.int32), n_found=_int32(1) + c["R"],
                O=torch.empty((H, N_q, D), dtype=dt, device="cuda"), lse=torch.empty((H, N_q), device="cuda"))


def _prepare_causal(c, gen, seed):
    H, N_q, dt = c["H"], c["q_frames"] * c["T"], _DTYPES[c["dtype"]]
    return dict(Q=_randn(gen, (H, N_q, D), dt), K_win=_randn(gen, (H, c["N_kv"], D), dt), V_win=_randn(gen, (H, c["N_kv"], D), dt),
                O=torch.empty((H, N_q, D), dtype=dt, device="cuda"),
                ws=_bytes(wk.wk_attention_block_causal_workspace_bytes(H, N_q)))


def _prepare_refresh(c, gen, seed):
    H, M, R, n, dt = c["H"], c["M"], c["R"], c["tokens"], _DTYPES[c["dtype"]]
    host = torch.empty((2, M, H, n, D), dtype=dt, pin_memory=True)
    host.copy_(_randn(gen, (2, M, H, n, D), dt))
    n_native, N_q = c["native_frames"] * c["T"], c["q_frames"] * c["T"]
    cap = n_native + R * n
    order = _ids(gen, M, R + 1)
    s = dict(store=wk.Store(list(host[0]), list(host[1])), wanted=(order[:R].clone(), torch.cat((order[:R - 1], order[R:])).contiguous()),
             slots=_int32(R) - 1, n_native=n_native, cap=cap, K_win=_randn(gen, (H, cap, D), dt), V_win=_randn(gen, (H, cap, D), dt),
             n_win=_int32(1), n_fetched=_int32(1), ws=_bytes(wk.wk_window_update_workspace_bytes(R)),
             Q=_randn(gen, (H, N_q, D), dt), O=torch.empty((2, H, N_q, D), dtype=dt, device="cuda"),
             att_ws=_attention_workspace(H, N_q, cap, dt), case=c)
    for ids in s["wanted"]:   # the rollout is under way: all chunks but the one that changes are resident
        _update(s, ids)
    return s


# ---- one pass -------------------------------------------------------------------------------------------------------

def run(state):
    return globals()["_run_" + state["case"]["kind"]](state, state["case"])


def _run_poses(s, c):
    wk.wk_score_chunks(s["poses"], c["M"], s["cur"], wk.WK_NORM_MAX, c["R"], s["ids"], s["dist"], s["n_found"])
    return s["ids"], s["dist"], s["n_found"]


def _run_step(s, c):
    wk.wk_compress_chunk(s["desc"], s["K"], s["V"], s["A"], s["kept"], s["K_out"], s["V_out"], s["ws"])
    _run_poses(s, c)
    wk.wk_gather_window(s["store"].desc, s["ids"], s["n_found"], c["R"], None, None, s["n_native"], s["K_win"], s["V_win"],
                        s["cap"], s["n_win"])
    wk.wk_attention(s["Q"], s["K_win"], s["V_win"], s["O"], None, N_kv=s["cap"], n_kv_dev=s["n_win"], workspace=s["att_ws"])
    return {k: s[k] for k in ("kept", "K_out", "V_out", "ids", "dist", "n_found", "K_win", "V_win", "n_win", "O")}


def _run_attention(s, c):
    wk.wk_attention(s["Q"], s["K_win"], s["V_win"], s["O"], s["lse"], N_kv=c["N_kv"], workspace=s["att_ws"])
    return s["O"], s["lse"]


def _run_compress(s, c):
    wk.wk_compress_chunk(s["desc"], s["K"], s["V"], None, s["kept"], s["K_out"], s["V_out"], s["ws"])
    return s["kept"], s["K_out"], s["V_out"], s["scores"]


def _run_query(s, c):
    wk.wk_chunk_lse(s["store"].desc, s["Q"], s["lse"])
    wk.wk_score_chunks_query(s["lse"], c["M"], c["H"] * c["N_q"], c["R"], s["ids"], s["mass"], s["n_found"], s["ws"])
    return s["lse"], s["ids"], s["mass"], s["n_found"]


def _run_in_place(s, c):
    wk.wk_attention_in_place(s["Q"], s["K_nat"], s["V_nat"], c["n_native"], s["store"].desc, s["ids"], s["n_found"], c["R"], s["O"], s["lse"])
    return s["O"], s["lse"]


def _run_causal(s, c):
    wk.wk_attention_block_causal(s["Q"], s["K_win"], s["V_win"], s["O"], c["row0"], c["T"], s["ws"])
    return s["O"]


def _update(s, ids):
    c = s["case"]
    wk.wk_window_update(s["store"].desc, ids, None, c["R"], c["tokens"], s["slots"], s["n_native"], s["K_win"], s["V_win"], s["cap"],
                        s["n_win"], s["n_fetched"], s["ws"])


def _run_refresh(s, c):
    for ids, O in zip(s["wanted"], s["O"]):
        _update(s, ids)
        wk.wk_attention(s["Q"], s["K_win"], s["V_win"], O, None, N_kv=s["cap"], n_kv_dev=s["n_win"], workspace=s["att_ws"])
    return {k: s[k] for k in ("slots", "n_win", "n_fetched", "K_win", "V_win", "O")}


# ---- what a pass cannot do without ------------------------------------------------------------------------------------

def _attention_work(H, N_q, N_kv, e, pairs=None):
    return 2.0 * H * D * e * (N_q + N_kv), 4.0 * H * D * (N_q * N_kv if pairs is None else pairs)


def _compress_work(c, batch, e):
    """K and the kept rows of V read, the kept rows of both written; two dot products per candidate (or the similarity
    product that the matrix-core form names) and the anchors' norms and mean."""
    desc = _compress_desc(c)
    n_out, _ = wk.wk_keep_count(desc.rho, desc.ratio_kind, desc.anchor_mode, c["F"], c["T"])
    ext = bool(c.get("external"))
    n_tok, n_cand = c["F"] * c["T"] + (c["T"] if ext else 0), (c["F"] - (0 if ext else 1)) * c["T"]
    per = 2.0 * c["T"] * n_cand if c.get("algo") == "gemm" else 4.0 * (n_cand + c["T"])
    return batch * c["H"] * D * e * (n_tok + 3.0 * n_out), batch * c["H"] * D * per, n_out


def work(case):
    c, kind = case, case["kind"]
    e = 4 if c.get("dtype") == "f32" else 2
    if kind == "poses":
        return {"bytes": 20.0 * c["M"] + 12.0 * c["R"], "flops": 100.0 * c["M"]}
    if kind == "step":
        b, f, n_out = _compress_work(c, 1, e)
        n_kv = c["native_frames"] * c["T"] + c["R"] * n_out
        ab, af = _attention_work(c["H"], c["q_frames"] * c["T"], n_kv, e)
        gather = 4.0 * c["R"] * n_out * c["H"] * D * e
        return {"bytes": b + ab + gather + 20.0 * c["M"], "flops": f + af}
    if kind == "attention":
        b, f = _attention_work(c["H"], c["N_q"], c["N_kv"], e)
    elif kind == "compress":
        b, f, _ = _compress_work(c, c["batch"], e)
    elif kind == "query":
        pairs = float(c["N_q"]) * c["M"] * c["tokens"]
        b = c["H"] * (D * e * (c["N_q"] + float(c["M"]) * c["tokens"]) + 8.0 * c["M"] * c["N_q"])
        f = 2.0 * c["H"] * D * pairs
    elif kind == "in_place":
        b, f = _attention_work(c["H"], c["N_q"], c["n_native"] + sum(_chunk_lengths(c)[:c["R"]]), e)
    elif kind == "causal":
        T, n = c["T"], c["q_frames"]
        hidden = T * T * n * (n - 1) // 2
        b, f = _attention_work(c["H"], n * T, c["N_kv"], e, n * T * c["N_kv"] - hidden)
    else:
        ab, af = _attention_work(c["H"], c["q_frames"] * c["T"], c["native_frames"] * c["T"] + c["R"] * c["tokens"], e)
        b, f = 2 * (ab + 4.0 * c["H"] * c["tokens"] * D * e), 2 * af
    return {"bytes": b, "flops": f}


def tolerance(case):
    """Selections, indices and copied rows are exact (no whole value may differ).  The bounds of floating results are four
    times what was measured against the same formulas in fp64, or between two orders of summation, over these ranges."""
    if case["kind"] == "poses":
        return {"rel": 1e-12}   # fp64 throughout
    if case["kind"] == "compress":
        return {"rel": 8e-7, "max": 3e-6}   # scores: fp32 partial sums of terms that cancel (measured 1.9e-7, 7.3e-7); rows are copied
    if case["kind"] == "query":
        return {"rel": 1e-4, "max": 1e-3}   # log-sum-exp over bf16-rounded weights (2.4e-5 at 300 keys, more at 64), and masses made of it
    if case.get("dtype") == "f32":
        return {"rel": 2.4e-5, "max": 1.3e-4}   # 100,000 products summed in fp32 (5.8e-6, 3.2e-5)
    return {"rel": 1.2e-2, "max": 6e-2}   # probabilities and output rounded to bf16 (2.9e-3, 1.5e-2)
