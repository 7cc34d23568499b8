#!/usr/bin/env python3
"""Writes wk_attn_loop_gfx950.inc and wk_attn_pair_loop_gfx950.inc: the steady-state loops of k_attn_bf16 (8 waves,
32 queries each, 64-key tiles) as hand-scheduled inline-assembly bodies for gfx950; and wk_attn_gap_loop_gfx950.inc and
wk_attn_gap_pair_loop_gfx950.inc, the same for windows that leave out a run of rows.

    python gen_attn_loop.py [directory]      (default: beside this script)

The loop does exactly what one trip of `step`s round the ring does in the C++ kernel -- four steps of one tile, or
two steps of a pair of tiles (kg = 2: wave group 0 takes the even tiles, group 1 the odd ones, through a group offset in
its LDS read addresses) -- the same ring protocol, the same arithmetic in the same order, but with the schedule fixed by hand
and without a running maximum:

  * probabilities are relative to a reference, the first tile's maximum, that moves only when a lane's row sum has reached 2^24 at the
    beginning of a trip: up by the power of two that brings the sum below 1, but by 2^63 at most.  Their size does not matter to bf16 or to the fp32 sums, so results
    are those of a running maximum up to rounding, and bit-identical where that does not move either.  Looking for the tiles' maxima was 23 of a
    step's 113 vector instructions.  What grows beyond fp32 within a trip leaves infinities or NaN in the sums, which the kernel looks for at the
    end (and then does its work once more in the compiled steps, with the running maximum);

  * K fragments are requested two pairs of reads ahead of the matrix instructions that consume them, V^T
    fragments six matrix instructions ahead; every wait on the LDS counter is partial (LDS reads return in
    order, so "at most n outstanding" names the read that has landed);
  * the softmax arithmetic of the tile being consumed (scale, exp2, round to bf16, row sum) is dealt evenly between the
    16 matrix instructions that form S^T of the next tile and the first of the 16 value products behind them, software-pipelined so
    that no instruction waits for its producer; a value product comes no earlier than the slot behind the last rounding it needs;
  * the last five value products of a step are kept back past the workgroup barrier and issued behind the next
    step's first K reads: they cover the latency of those reads, which cannot be requested before the barrier;
  * tile loads (global memory -> LDS) are issued from here, so the compiler's wait-count pass never sees them.

With a gap, the tile that holds the first row behind it is loaded by code behind the loop, which moves the lanes whose rows lie
behind it, and then the cursor.  Its step is found by counting, one scalar comparison and branch a step: comparing the cursor at
every tile load instead made the loop 2.5 % slower.

Hazards the assembler does not resolve, and how the schedule respects them: a register written by a matrix
instruction is read by vector instructions only many matrix instructions later (S^T is read a step later, behind the step's first 11 value
products; the rare rescale of O^T waits 16 states first); a v_exp result is consumed at least three instructions later; v_mov ->
v_permlane32_swap has two wait states between.

Register map (VGPR), fixed through operand constraints in the kernel source:
  O   v[0:63]     o[b] = v[16b : 16b+15]
  SA  v[64:95]    S^T tile at even ring positions (two 32-key blocks of 16 registers)
  SB  v[96:127]   ... at odd ring positions
  Q   v[128:159]  qb[st] = v[128+4st : 131+4st]
  P   v[160:175]  pb[ks] = v[160+4ks : 163+4ks]
  KF  v[176:199]  six K fragment buffers
  VF  v[200:223]  six V^T fragment buffers (two 8-byte transpose reads each)
  KAD v[224:231]  LDS address of K operand read st
  VAD v[232:235]  LDS address of V^T operand read blk (V ring base included)
  KSRC v[236:237] VSRC v[238:239]   per-lane source offsets of this wave's tile loads
  M v240  L v[241:242]   reference (log2 units), row sums of the even and the odd tiles (kg = 2: of this wave group's tiles, and
              nothing)
  T   v[244:245]  temporaries
SGPR:
  s[36:37], s[38:39] the K tile and the V tile requested next (with a gap: K and V rows of this head, and s40, s41 their byte offsets),
  s42 LDS address of this wave's share of K ring slot 0, s43 scale*log2(e), s44 groups left, s45 the caller's m0;
  with a gap: s46 byte offset, gap left out, of the first row behind it, s47 bytes of the gap, s48 cursor of the tile that
  holds that row, s49 steps left in front of the one that requests this K tile (its V tile comes one later), and two
"""
import os
import sys

TILE = 16384          # bytes of one 64-key K or V tile
VRING = 65536         # the V ring sits behind the four K slots
DEFER = 5             # value products kept back past the barrier (with scalar tile cursors: LingBot window 2,224 -> 2,214 us with 3, 2,208 with 5;
                      # vector work beside them too: 2,228 to 2,249)

S = {0: 64, 1: 96}


def Q(st):
    return 128 + 4 * st


def P(ks):
    return 160 + 4 * ks


def KF(i):
    return 176 + 4 * i


def VF(i):
    return 200 + 4 * i


def KAD(st):
    return 224 + st


def VAD(b):
    return 232 + b


KSRC, VSRC = (236, 237), (238, 239)
M = 240
L = (241, 242)
T0, T1 = 244, 245
ONES = "0x3f803f80"    # two bf16 ones
GROWN = "0x4b800000"   # 2^24
VECTOR_SLOTS = 22      # matrix instructions that a step's vector work is dealt over (LingBot window 2,184 us with 16, 2,178 with 20, 2,155 with 22, 2,158 with 24)


def rng(a, n):
    return f"v[{a}:{a + n - 1}]"


class Emitter:
    """Collects instructions and keeps the queue of outstanding LDS reads, from which the partial waits follow."""

    def __init__(self):
        self.lines = []
        self.lds = []
        self.next_id = 0
        self.deferred = []
        self.behind = []     # code behind the loop

    def emit(self, s):
        self.lines.append(s)

    def lds_read(self, text):
        self.emit(text)
        self.lds.append(self.next_id)
        self.next_id += 1
        assert len(self.lds) <= 15, "the 4-bit LDS counter would saturate"
        return self.next_id - 1

    def wait_for(self, rid):
        if rid in self.lds:
            k = self.lds.index(rid)
            self.emit(f"s_waitcnt lgkmcnt({len(self.lds) - 1 - k})")
            self.lds = self.lds[k + 1:]


def head(E, pos, kg):
    """The first three pairs of K fragment reads of a step (the wave's next tile, kg ring slots on)."""
    koff = ((pos + kg) & 3) * TILE
    kreads = {}
    for st in range(3):
        for b in range(2):
            buf = (2 * st + b) % 6
            rid = E.lds_read(f"ds_read_b128 {rng(KF(buf), 4)}, v{KAD(st)} offset:{koff + b * 8192}")
            kreads[(st, b)] = (buf, rid)
    return kreads


def step(E, pos, kg, kreads=None, gap=False):
    cur = S[(pos // kg) & 1]          # S^T of the tile consumed in this step (ring slot pos)
    nxt = S[(pos // kg + 1) & 1]      # S^T of the wave's next tile, formed in this step
    koff = ((pos + kg) & 3) * TILE
    voff = pos * TILE

    if kreads is None:
        kreads = head(E, pos, kg)
        for txt in E.deferred:   # the value products kept back by the previous step
            E.emit(txt)
        E.deferred = []

    def issue_k(st):
        for b in range(2):
            buf = (2 * st + b) % 6
            rid = E.lds_read(f"ds_read_b128 {rng(KF(buf), 4)}, v{KAD(st)} offset:{koff + b * 8192}")
            kreads[(st, b)] = (buf, rid)

    # this wave's share of the K tiles requested in this step (into the slots whose tiles went into S^T one step ago)
    # and of the V tiles (into the slots behind the ones read in this step)
    def load(cursor, base, src, slots):
        for slot in slots:
            for i in range(2):
                E.emit(f"s_add_u32 m0, s42, {slot + i * 1024}")
                if gap:
                    E.emit(f"v_add_u32_e32 v{T0}, {cursor}, v{src[i]}")
                    E.emit(f"global_load_lds_dwordx4 v{T0}, {base}")
                else:   # the scalar base is the cursor: no vector instruction
                    E.emit("s_nop 0")   # (m0's wait state)
                    E.emit(f"global_load_lds_dwordx4 v{src[i]}, {base}")
            if gap:
                E.emit(f"s_add_u32 {cursor}, {cursor}, {TILE}")
            else:
                lo, hi = base[2:-1].split(":")
                E.emit(f"s_add_u32 s{lo}, s{lo}, {TILE}")
                E.emit(f"s_addc_u32 s{hi}, s{hi}, 0")

    def load_at_gap(name, cursor, base, src, slots):
        for t, slot in enumerate(slots):
            lab = f"{name}{pos + t}_%="
            E.behind += [f"s_cmp_lg_u32 {cursor}, s48", f"s_cbranch_scc1 L_plain_{lab}"]
            for lanes in (True, False):
                for i in range(2):
                    E.behind += [f"s_add_u32 m0, s42, {slot + i * 1024}", f"v_add_u32_e32 v{T0}, {cursor}, v{src[i]}"]
                    if lanes:
                        E.behind += [f"v_cmp_le_u32_e32 vcc, s46, v{T0}", f"v_mov_b32_e32 v{T1}, s47",
                                     f"v_cndmask_b32_e32 v{T1}, 0, v{T1}, vcc", f"v_add_u32_e32 v{T0}, v{T0}, v{T1}"]
                    E.behind += [f"global_load_lds_dwordx4 v{T0}, {base}"]
                if lanes:
                    E.behind += [f"s_add_u32 {cursor}, {cursor}, s47", f"s_branch L_next_{lab}", f"L_plain_{lab}:"]
            E.behind += [f"L_next_{lab}:", f"s_add_u32 {cursor}, {cursor}, {TILE}"]

    loads = (("k", "s40", "s[36:37]", KSRC, [(pos + t) * TILE for t in range(kg)]),
             ("v", "s41", "s[38:39]", VSRC, [VRING + ((pos + 3 - (kg - 1) + t) & 3) * TILE for t in range(kg)]))
    if gap:
        E.emit("s_sub_u32 s49, s49, 1")
        E.emit("s_cmp_lt_u32 s49, 2")
        E.emit(f"s_cbranch_scc1 L_gap_{pos}_%=")
        E.behind.append(f"L_gap_{pos}_%=:")
        for args in loads:
            load_at_gap(*args)
        E.behind.append(f"s_branch L_loaded_{pos}_%=")
    for _, *args in loads:
        load(*args)
    if gap:
        E.emit(f"L_loaded_{pos}_%=:")

    if pos == 0:   # (O^T is complete here, and the tile consumed next still holds its scores)
        E.emit(f"v_add_f32_e32 v{T0}, v{L[0]}, v{L[1]}")
        E.emit(f"v_cmp_ngt_f32_e32 vcc, {GROWN}, v{T0}")   # (true of NaN)
        E.emit("s_cbranch_vccnz L_grown_%=")
        E.emit("L_weighed_%=:")
        # (the exponent of an infinity and of NaN reads as 0.  63 at most: v_exp gives 0 below -126, which would leave out all keys so far, and the reference
        # plus e, rounded, is up to e further away than e)
        E.behind += ["L_grown_%=:", "s_nop 7", "s_nop 7", f"v_frexp_exp_i32_f32_e32 v{T0}, v{T0}", f"v_mov_b32_e32 v{T1}, v{T0}", "s_nop 1",
                     f"v_permlane32_swap_b32_e32 v{T0}, v{T1}", "s_nop 0", f"v_max3_i32 v{T0}, v{T0}, v{T1}, 0", f"v_min_i32_e32 v{T0}, 63, v{T0}",
                     f"v_cvt_f32_i32_e32 v{T0}, v{T0}",
                     f"v_add_f32_e32 v{T0}, v{M}, v{T0}", f"v_sub_f32_e32 v{T1}, v{M}, v{T0}", f"v_exp_f32_e32 v{T1}, v{T1}", f"v_mov_b32_e32 v{M}, v{T0}",
                     "s_nop 1"]
        E.behind += [f"v_mul_f32_e32 v{L[t]}, v{L[t]}, v{T1}" for t in range(2)]
        E.behind += [f"v_mul_f32_e32 v{r}, v{T1}, v{r}" for r in range(64)]
        E.behind.append("s_branch L_weighed_%=")

    # softmax arithmetic of the tile consumed, in place in its registers; element e is register cur + e.
    # Slot i: scale elements 2i, 2i+1; exp2 of the pair scaled one slot ago; round the pair exponentiated one slot
    # ago into P; add the pair rounded one slot ago to the row sum.
    slots = [[] for _ in range(32)]   # behind each of the step's matrix instructions
    groups = 16 + 3
    place = [i * (VECTOR_SLOTS - 1) // (groups - 1) for i in range(groups)]
    for i in range(groups):
        ops = []
        if i < 16:
            ops += [f"v_fma_f32 v{cur + 2 * i}, v{cur + 2 * i}, s43, -v{M}",
                    f"v_fma_f32 v{cur + 2 * i + 1}, v{cur + 2 * i + 1}, s43, -v{M}"]
        if 1 <= i < 17:
            k = i - 1
            ops += [f"v_exp_f32_e32 v{cur + 2 * k}, v{cur + 2 * k}", f"v_exp_f32_e32 v{cur + 2 * k + 1}, v{cur + 2 * k + 1}"]
        if 2 <= i < 18:
            k = i - 2
            ops += [f"v_cvt_pk_bf16_f32 v{P(0) + k}, v{cur + 2 * k}, v{cur + 2 * k + 1}"]
        if 3 <= i < 19:
            ops += [f"v_dot2c_f32_bf16_e32 v{L[0 if kg == 2 else pos & 1]}, {ONES}, v{P(0) + i - 3}"]
        slots[place[i]] += ops
    assert all(place[4 * ks + 3 + 2] < 16 + 4 * ks for ks in range(4))   # rounded before step ks of the value product

    vreads = {}

    def issue_v(n):
        ks, b = n // 4, n % 4
        buf = n % 6
        E.lds_read(f"ds_read_b64_tr_b16 {rng(VF(buf), 2)}, v{VAD(b)} offset:{voff + ks * 4096}")
        rid = E.lds_read(f"ds_read_b64_tr_b16 {rng(VF(buf) + 2, 2)}, v{VAD(b)} offset:{voff + ks * 4096 + 2048}")
        vreads[n] = (buf, rid)

    # S^T of the next tile: K block b (32 keys) x 16 features of step st, the two blocks' chains alternating
    for st in range(8):
        for b in range(2):
            buf, rid = kreads[(st, b)]
            E.wait_for(rid)
            c = "0" if st == 0 else rng(nxt + 16 * b, 16)
            E.emit(f"v_mfma_f32_32x32x16_bf16 {rng(nxt + 16 * b, 16)}, {rng(KF(buf), 4)}, {rng(Q(st), 4)}, {c}")
            for op in slots[2 * st + b]:
                E.emit(op)
        if st + 3 < 8:
            issue_k(st + 3)
        if st >= 5:   # the first V^T fragments, while the last K fragments are consumed
            issue_v(2 * (st - 5))
            issue_v(2 * (st - 5) + 1)
    # O^T += V^T P^T: feature block b x 16 keys of step ks
    for n in range(16):
        ks, b = n // 4, n % 4
        buf, rid = vreads[n]
        E.wait_for(rid)
        txt = f"v_mfma_f32_32x32x16_bf16 {rng(16 * b, 16)}, {rng(VF(buf), 4)}, {rng(P(ks), 4)}, {rng(16 * b, 16)}"
        if n >= 16 - DEFER:
            E.deferred.append(txt)
        else:
            E.emit(txt)
        if n + 6 < 16:
            issue_v(n + 6)
        for op in slots[16 + n]:
            E.emit(op)
    assert not E.lds
    # kg = 1: all but the tile loads of this step and the one before have landed; kg = 2: all have
    E.emit(f"s_waitcnt vmcnt({8 if kg == 1 else 0})")
    E.emit("s_barrier")


def generate(kg=1, gap=False):
    # what the last step of a trip keeps back is the same text in every iteration: find it with a dry run
    dry = Emitter()
    for pos in range(0, 4, kg):
        step(dry, pos, kg, gap=gap)
    carried = list(dry.deferred)

    E = Emitter()
    E.emit("s_mov_b32 s45, m0")   # m0 is the compiler's to manage: hand it back as it was
    # entry: the first reads of position 0 with nothing kept back (the C++ step before finished its tile)
    kr = head(E, 0, kg)
    E.emit("s_branch L_body_%=")
    state = (list(E.lds), E.next_id)
    E.emit("L_group_%=:")
    E.lds, E.next_id = [], 0
    assert head(E, 0, kg) == kr and (list(E.lds), E.next_id) == state
    for txt in carried:
        E.emit(txt)
    E.emit("L_body_%=:")
    step(E, 0, kg, kreads=kr, gap=gap)
    for pos in range(kg, 4, kg):
        step(E, pos, kg, gap=gap)
    assert E.deferred == carried
    E.emit("s_sub_u32 s44, s44, 1")
    E.emit("s_cmp_lg_u32 s44, 0")
    E.emit("s_cbranch_scc1 L_group_%=")
    for txt in carried:
        E.emit(txt)
    E.emit("s_nop 7")    # the compiler's code behind the block may read O^T at once
    E.emit("s_nop 7")
    E.emit("s_mov_b32 m0, s45")
    E.emit("s_branch L_end_%=")
    E.lines += E.behind
    E.emit("L_end_%=:")
    return E.lines


def render(kg=1, gap=False):
    out = ["// Written by gen_attn_loop.py: the hand-scheduled steady-state loop of k_attn_bf16 (see that script).\n"]
    out += ['"' + ln + '\\n\\t"\n' for ln in generate(kg, gap)]
    return "".join(out)


FILES = {1: "wk_attn_loop_gfx950.inc", 2: "wk_attn_pair_loop_gfx950.inc"}
GAP_FILES = {1: "wk_attn_gap_loop_gfx950.inc", 2: "wk_attn_gap_pair_loop_gfx950.inc"}

if __name__ == "__main__":
    here = sys.argv[1] if len(sys.argv) > 1 else os.path.dirname(os.path.abspath(__file__))
    for gap, files in enumerate((FILES, GAP_FILES)):
        for kg, name in files.items():
            with open(os.path.join(here, name), "w") as f:
                f.write(render(kg, bool(gap)))
            print(os.path.join(here, name))
