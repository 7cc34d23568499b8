#!/usr/bin/env python3
"""Writes wk_lse_loop_gfx950.inc: the steady-state loop of k_lse_wide_bf16 (4 waves, 64 queries each, 64-key tiles, no
value product) as a hand-scheduled inline-assembly body for gfx950.

    python gen_lse_loop.py [directory]      (default: beside this script)

A trip is two steps; the loop may end behind the first.  A step forms S^T of the next tile -- 32 matrix instructions, first the tile's keys 0..31 against both
32-query blocks, then keys 32..63 -- and turns S^T of the current one into the row sums: scale and subtract the reference, exp2,
round to bf16, add.  Every K fragment read from LDS feeds two matrix instructions.  The vector work of a step is dealt evenly over a window of 32
matrix instructions that begins three instructions behind the step's first, because the current tile's last products come right
before: neither pipe is full, and the vector pipe, which is the busier one, must not idle.  The last four matrix instructions of a step are kept back past
the workgroup barrier, together with the vector work that belongs beside them, and cover the latency of the next step's
first K reads.  A v_exp result is used six
instructions later, a row sum is read four behind its last v_dot2c (no hardware wait).

Register map (VGPR), fixed through operand constraints in the kernel source:
  X v[0:63]  Y v[64:127]   S^T of tiles at even / odd steps: key block kb, query block q at 32*kb + 16*q
  Q  v[128:191]  B operand of query block q, step st at 32*q + 4*st
  KF v[192:223]  eight K fragment buffers
  KAD v[224:231] LDS address of K operand read st, in the ring half of the step's current tile
  KSRC v[232:235]  source offsets, in a tile, of this wave's four loads
  M v[240:241]  L v[242:245]  reference (log2 units) of query block q; row sums of even / odd tiles at 2*parity + q
  PK v[246:247]  rounded pairs; LIMIT v[248:249] 2^8 above the row sums before the tile; T v[250:251] temporaries
SGPR:
  s[36:39] the K rows of this head from the tile requested next on, as a buffer, s42 LDS address of this wave's share of the slot
  it goes to, s43 scale*log2(e), s44 steps left but one, s45 the caller's m0, s[46:47] a comparison's
  lanes, s48 and s49 what brings the read addresses and s42 to the other half of the ring
"""
import os
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, HERE)
from gen_attn_loop import Emitter, ONES, TILE, rng  # noqa: E402

SLOTS = 32            # matrix instructions of a step
BACK = 4              # of them kept back past the barrier
LEAD = 3              # matrix instructions of a step in front of its own vector work
AHEAD = 5             # K fragments requested ahead of the one in use
S = {0: 0, 1: 64}
M, L, PK, LIMIT, T = 240, 242, 246, 248, 250
GROWN = "0x43800000"         # 2^8
MINUS_ONES = "0xbf80bf80"    # two bf16
KSRC, KAD = 232, 224


def Q(q, st):
    return 128 + 32 * q + 4 * st


def KF(n):
    return 192 + 4 * (n % 8)


def read_fragment(E, n, off):
    kb, st = n // 8, n % 8
    return E.lds_read(f"ds_read_b128 {rng(KF(n), 4)}, v{KAD + st} offset:{off + kb * 8192}")


def product(nxt, i):
    n, q = i // 2, i & 1   # a fragment feeds two products; the accumulation chains alternate
    kb, st = n // 8, n % 8
    d = nxt + 32 * kb + 16 * q
    return f"v_mfma_f32_32x32x16_bf16 {rng(d, 16)}, {rng(KF(n), 4)}, {rng(Q(q, st), 4)}, {'0' if st == 0 else rng(d, 16)}"


def sums(tile, par):
    """Scale, exp2, round to bf16 and sum, pair by pair, software-pipelined; the weights stay in their registers."""
    pairs = [(tile + 32 * kb + 16 * q + 2 * e, q) for kb in range(2) for e in range(8) for q in range(2)]
    ops = [f"v_add_f32_e32 v{LIMIT + q}, {GROWN}, v{L + 2 * par + q}" for q in range(2)]
    for i in range(len(pairs) + 3):
        if i < len(pairs):
            r, q = pairs[i]
            ops += [f"v_fma_f32 v{r}, v{r}, s43, -v{M + q}", f"v_fma_f32 v{r + 1}, v{r + 1}, s43, -v{M + q}"]
        if 1 <= i < len(pairs) + 1:
            r, _ = pairs[i - 1]
            ops += [f"v_exp_f32_e32 v{r}, v{r}", f"v_exp_f32_e32 v{r + 1}, v{r + 1}"]
        if 2 <= i < len(pairs) + 2:
            r, _ = pairs[i - 2]
            ops += [f"v_cvt_pk_bf16_f32 v{PK + i % 2}, v{r}, v{r + 1}"]
        if i == 19:   # the first key block's sums are complete
            ops += compare(par)
        if i >= 3:
            r, q = pairs[i - 3]
            ops += [f"v_dot2c_f32_bf16_e32 v{L + 2 * par + q}, {ONES}, v{PK + (i - 1) % 2}"]
        if i == 20:
            ops += ["\n".join(grown(par, 0, ""))]
    return ops


def compare(par):
    return [f"v_cmp_ge_f32_e32 vcc, v{L + 2 * par}, v{LIMIT}", f"v_cmp_ge_f32_e64 s[46:47], v{L + 2 * par + 1}, v{LIMIT + 1}"]


BEHIND = {}   # code behind the loop, which itself takes no branch but its own


def grown(par, kb, tag):
    """Behind a key block's sums: where a lane's sum over the tile reached 2^8, what the weights lost in rounding is added after
    all; behind the tile's second block the reference then goes up by the power of two that brings the row sums back to
    about 1."""
    name = f"L_same_{par}{kb}{tag}"
    ops = [f"L_grown_{par}{kb}{tag}_%=:"]
    for q in range(2):
        l, r = L + 2 * par + q, S[par] + 32 * kb + 16 * q
        ops += [f"v_cmp_ge_f32_e32 vcc, v{l}, v{LIMIT + q}", f"s_cbranch_vccz {name}_{q}_%="]
        for e in range(8):
            ops += [f"v_cvt_pk_bf16_f32 v{T}, v{r + 2 * e}, v{r + 2 * e + 1}", f"v_add_f32_e32 v{T + 1}, v{r + 2 * e}, v{r + 2 * e + 1}",
                    f"v_dot2c_f32_bf16_e32 v{T + 1}, {MINUS_ONES}, v{T}", "s_nop 3", f"v_add_f32_e32 v{l}, v{l}, v{T + 1}"]
        if kb == 1:
            ops += [f"v_sub_f32_e32 v{T}, v{l}, v{LIMIT + q}", f"v_add_f32_e32 v{T}, {GROWN}, v{T}", f"v_frexp_exp_i32_f32_e32 v{T}, v{T}",
                    f"v_add_u32_e32 v{T}, -5, v{T}", f"v_mov_b32_e32 v{T + 1}, v{T}",
                    "s_nop 1", f"v_permlane32_swap_b32_e32 v{T}, v{T + 1}", "s_nop 0", f"v_max_i32_e32 v{T}, v{T}, v{T + 1}",
                    f"v_max_i32_e32 v{T}, 0, v{T}", f"v_cvt_f32_i32_e32 v{T + 1}, v{T}", f"v_add_f32_e32 v{M + q}, v{M + q}, v{T + 1}",
                    f"v_sub_u32_e32 v{T}, 0, v{T}", f"v_ldexp_f32 v{L + q}, v{L + q}, v{T}", f"v_ldexp_f32 v{L + 2 + q}, v{L + 2 + q}, v{T}"]
        ops += [f"{name}_{q}_%=:"]
    BEHIND[name] = ops + [f"s_branch {name}_%="]
    return ["s_or_b64 vcc, vcc, s[46:47]", f"s_cbranch_scc1 L_grown_{par}{kb}{tag}_%=", f"{name}_%=:"]


def load(i, par):
    # (a buffer that begins at the tile and ends with the window: rows past its end, which would have to be clamped lane by lane, read as 0:
    # a step's eight vector instructions for its loads are none.  40 chunks of 1,560 keys x 40 heads x 4,680 queries 2,852 -> 2,821 us, 60 of 880 x 12 x 2,640 433 -> 429)
    return "\n".join([f"s_add_u32 m0, s42, {par * TILE + i * 1024}", "s_nop 0", f"buffer_load_dwordx4 v{KSRC + i}, s[36:39], 0 offen lds"])


def vector_work(par):
    """The vector work of a step, dealt over its 32-instruction window: window[k] goes behind the k-th matrix instruction of
    it (k = 0 is the step's instruction LEAD)."""
    ops = sums(S[par], par)
    window = [[] for _ in range(SLOTS)]
    for k, op in enumerate(ops):
        window[k * len(window) // len(ops)].append(op)
    for i in range(4):
        window[1 + 2 * i].append(load(i, par))
    # behind the step's last K read: the addresses of the other half of the ring for the next step
    if par == 0:
        for st in range(8):
            window[SLOTS - BACK - LEAD - 1 - st // 4].append(f"v_add_u32_e32 v{KAD + st}, s48, v{KAD + st}")
    window[8] += [f"s_add_u32 s36, s36, {TILE}", "s_addc_u32 s37, s37, 0", f"s_sub_u32 s38, s38, {TILE}", "s_cselect_b32 s38, 0, s38"]   # (not below 0)
    if par == 1:
        window[8] += ["s_add_u32 s42, s42, s49", "s_sub_u32 s48, 0, s48", "s_sub_u32 s49, 0, s49"]
    return window


def emit_all(E, ops):
    for op in ops:
        for ln in op.split("\n"):
            E.emit(ln)


def finish(E, par, carried, lead, tag=""):
    """What step par kept back, beside the products in `lead` (callables) of the step behind it."""
    products, window = carried
    for put, ops in zip([lambda txt=txt: E.emit(txt) for txt in products] + lead, window):
        put()
        emit_all(E, ops)
    emit_all(E, ["s_nop 3"] + compare(par) + grown(par, 1, tag))


def lead_in(E, par, carried):
    """A step's first K reads, what the step before kept back, and the step's first LEAD matrix instructions."""
    off = TILE if par == 0 else 0
    rid = {n: read_fragment(E, n, off) for n in range(AHEAD)}

    def put(i):
        E.wait_for(rid[i // 2])
        E.emit(product(S[par ^ 1], i))
        if i % 2 == 1 and i // 2 + AHEAD < 16:
            rid[i // 2 + AHEAD] = read_fragment(E, i // 2 + AHEAD, off)

    lead = [lambda i=i: put(i) for i in range(LEAD)]
    if carried is not None:
        finish(E, par ^ 1, carried, lead)
    else:
        for f in lead:
            f()
    return rid


def body(E, par, rid):
    off = TILE if par == 0 else 0
    window = vector_work(par)
    for i in range(LEAD, SLOTS - BACK):
        E.wait_for(rid[i // 2])
        E.emit(product(S[par ^ 1], i))
        if i % 2 == 1 and i // 2 + AHEAD < 16:
            rid[i // 2 + AHEAD] = read_fragment(E, i // 2 + AHEAD, off)
        emit_all(E, window[i - LEAD])
    E.wait_for(rid[15])
    assert not E.lds
    E.emit("s_waitcnt vmcnt(8)")   # all but the tile loads of this step and the one before have landed
    E.emit("s_barrier")
    return [product(S[par ^ 1], i) for i in range(SLOTS - BACK, SLOTS)], window[SLOTS - BACK - LEAD:]


def generate():
    dry = Emitter()
    body(dry, 0, lead_in(dry, 0, None))
    carried = body(dry, 1, lead_in(dry, 1, None))

    E = Emitter()
    def end():
        E.emit("s_nop 7")    # the compiler's code behind the block may read S^T at once
        E.emit("s_nop 7")
        E.emit("s_mov_b32 m0, s45")

    E.emit("s_mov_b32 s45, m0")   # m0 is the compiler's to manage: handed back as it was
    E.emit("s_mov_b32 s48, 0x8000")
    E.emit("s_mov_b32 s49, 0x8000")
    rid = lead_in(E, 0, None)
    state = list(E.lds)
    E.emit("s_branch L_body_%=")
    # Where one wave per SIMD runs, the trip's place in a 32-byte fetch matters: 3 heads x 300 queries x 211,200 keys 2.90 ms
    # with 4 or 16 bytes in front of it, 2.98 with 0 or 20 (12 x 880 x 21,120: 296 and 304 us).
    E.emit(".p2align 6")
    E.emit("s_nop 0")
    E.emit("L_trip_%=:")
    E.lds, E.next_id = [], 0
    assert lead_in(E, 0, carried) == rid and E.lds == state
    E.emit("L_body_%=:")
    kept = body(E, 0, rid)
    E.emit("s_sub_u32 s44, s44, 1")
    E.emit("s_cbranch_scc1 L_odd_%=")
    assert body(E, 1, lead_in(E, 1, kept)) == carried
    E.emit("s_sub_u32 s44, s44, 1")
    E.emit("s_cbranch_scc0 L_trip_%=")
    finish(E, 1, carried, [lambda: None] * LEAD, "e")
    end()
    E.emit("s_branch L_end_%=")
    E.emit("L_odd_%=:")    # S^T of the last tile is in Y
    finish(E, 0, kept, [lambda: None] * LEAD, "o")
    end()
    for r in range(64):
        E.emit(f"v_mov_b32_e32 v{S[0] + r}, v{S[1] + r}")
    E.emit("s_branch L_end_%=")
    for ops in BEHIND.values():
        emit_all(E, ops)
    E.emit("L_end_%=:")
    return E.lines


def render():
    out = ["// Written by gen_lse_loop.py: the hand-scheduled steady-state loop of k_lse_wide_bf16 (see that script).\n"]
    out += ['"' + ln + '\\n\\t"\n' for ln in generate()]
    return "".join(out)


NAME = "wk_lse_loop_gfx950.inc"

if __name__ == "__main__":
    path = os.path.join(sys.argv[1] if len(sys.argv) > 1 else HERE, NAME)
    with open(path, "w") as f:
        f.write(render())
    print(path)
