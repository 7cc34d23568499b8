// Attention of the denoising chunk's queries over the assembled KV window (paper Sec. 4.2,
// Sec. 4.3): O = softmax(Q K^T * scale) V per head, every window key visible.
//
// Both kernels (bf16 and fp32) use the same transposed formulation, chosen for the CDNA
// 32x32 MFMA register layout (lane l of a wave owns column l%32 of the 32x32 result and
// rows 8*(r/4) + 4*(l/32) + r%4 for accumulator register r):
//
//     S^T = K  Q^T     A operand = K rows (from LDS),     B operand = Q^T (registers, loaded once)
//     O^T = V^T P^T    A operand = V^T    (from LDS),     B operand = P^T (registers)
//
// In S^T a lane's column is one query, so the online-softmax row statistics are per-lane scalars:
// the row max needs one exchange between lane l and lane l+32, the row sum none until the end,
// and the rescale factor of O^T is again a per-lane scalar.  The S^T accumulator registers are,
// after exp2 and rounding, exactly the B operand of the second product: which key an MFMA
// "k slot" means is a free choice, as long as the V^T operand uses the same choice.
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <type_traits>

#include "wk_internal.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short i16x8 __attribute__((ext_vector_type(8)));

struct AttnArgs {
    const char *Q;
    const char *K;
    const char *V;
    char *O;
    float *lse;
    int H, N_q, N_kv, kv_row_stride;
    float scale_log2;  // scale * log2(e): softmax is evaluated with exp2
    const int32_t *n_kv_dev;
    int n_qtiles;
    int per_xcd;       // work items per XCD in the launch order
    int splits;        // key-range splits per (head, query tile); 1 = none
    float *part_o;     // splits > 1: [splits][H][N_q][128] unnormalised fp32 partial outputs
    float *part_ml;    //             [splits][H][N_q][2] running max (log2 units) and row sum
    // batch over stored chunks (log-sum-exp only): chunk c has keys k_table[c] = [H][n_tok[c]][128]
    // and writes lse + c*H*N_q.  n_chunks = 0: one window, K above.
    const void *const *k_table;
    const int32_t *n_tok;
    int n_chunks;
    // a launch may cover queries [q_off, q_off + N_q) of arrays that hold q_rows rows per head
    // (Q, O, lse and the partial results), and a key range that starts kv_start rows into the
    // window (only used to convert *n_kv_dev); part_slot >= 0 makes it write its (O, max, sum)
    // as split `part_slot` for k_attn_merge instead of a final result.
    int q_rows, q_off, kv_start, part_slot;
    // rows [gap_row, gap_row + gap_len) of the window are not part of it (k_attn_bf16<.., GAP>)
    int gap_row = 0, gap_len = 0;
    // attention in place over the store (k_attn_bf16<.., IN_PLACE>): the window is K/V above (N_kv native
    // rows, may be 0) followed by the stored chunks ids[0 .. min(*n_ids, R_max)), read where they are
    // stored: chunk c has keys k_table[c] and values v_table[c], both [H][n_tok[c]][128].
    const void *const *v_table;
    const int32_t *ids;
    const int32_t *n_ids;
    int R_max, store_M;
    // host-known upper bound of n_tok[] (store descriptors): a chunk that claims more rows is treated as
    // absent, so no length the host has not seen can reach the 32-bit byte offsets of the tile loads
    int max_tok;
};

// bf16 tile loads form 32-bit byte offsets of rows (256 B each), up to four tiles past the last one
constexpr int kMaxRowsBf16 = (1 << 24) - 512;

constexpr int kXcds = 8;

// Workgroups are handed to the 8 XCDs round-robin by their linear id.  Work items are numbered
// head-major (all query tiles of head 0, then head 1, ...); giving XCD x the contiguous range
// [x*per_xcd, (x+1)*per_xcd) keeps the query tiles that stream the same head's K/V on one XCD,
// so that head's window is fetched from HBM once into that XCD's L2 instead of once per tile.
// With a split key range the items of one head are ordered split-major, so the query tiles that
// stream the same slice of K/V stay neighbours.  A batch over stored chunks (one key range each)
// is ordered head, chunk, query tile: a head's queries stay in the XCD's L2 while the chunks' keys
// stream through once.
__device__ inline bool work_item(const AttnArgs &a, int &c, int &h, int &qt, int &sp) {
    const int lin = blockIdx.x;
    const int w = (lin % kXcds) * a.per_xcd + lin / kXcds;
    if (lin / kXcds >= a.per_xcd) return false;
    if (a.n_chunks > 0) {
        const int per_head = a.n_chunks * a.n_qtiles;
        if (w >= a.H * per_head) return false;
        h = w / per_head;
        c = (w % per_head) / a.n_qtiles;
        qt = w % a.n_qtiles;
        sp = 0;
        return true;
    }
    if (w >= a.H * a.n_qtiles * a.splits) return false;
    c = 0;
    h = w / (a.n_qtiles * a.splits);
    const int rem = w % (a.n_qtiles * a.splits);
    sp = rem / a.n_qtiles;
    qt = rem % a.n_qtiles;
    return true;
}

// Several launches folded into one grid (used by the frame-causal entry point): each entry is what
// one plain launch would have been told -- which queries, which key range, which partial slot -- and which rows to leave out.
// Work items are numbered head-major over all entries, so a head's entries share an XCD.
struct SubLaunch { int q_off, N_q, n_qtiles, kv_off, N_kv, kv_start, part_slot, gap_row, gap_len; };
constexpr int kMaxSub = 8;
struct SubTable { int n, per_head; SubLaunch s[kMaxSub]; };

// MULTI: pick this workgroup's entry and make the (by-value) arguments look like that launch.
template <bool MULTI>
__device__ inline bool select_work(AttnArgs &a, const SubTable &t, size_t row_bytes, int &c, int &h, int &qt,
                                   int &sp);

// The window this workgroup reads: its keys, row stride between heads and length; where lse goes.
struct Window {
    const char *K;
    float *lse;
    int stride, n_kv;
};

__device__ inline Window window_of(const AttnArgs &a, int c) {
    Window w;
    if (a.n_chunks > 0) {
        w.K = reinterpret_cast<const char *>(a.k_table[c]);
        w.n_kv = w.stride = a.n_tok[c];
        if (w.n_kv > a.max_tok) w.n_kv = 0;   // violates the descriptor's bound: holds no token
        w.lse = a.lse + (size_t)c * a.H * a.q_rows;
    } else {
        w.K = a.K;
        w.stride = a.kv_row_stride;
        w.lse = a.lse;
        w.n_kv = a.N_kv;
        if (a.n_kv_dev) {
            const int m = *a.n_kv_dev - a.kv_start;
            w.n_kv = m < w.n_kv ? m : w.n_kv;
        }
    }
    if (w.n_kv < 0) w.n_kv = 0;
    return w;
}

template <bool MULTI>
__device__ inline bool select_work(AttnArgs &a, const SubTable &t, size_t row_bytes, int &c, int &h, int &qt,
                                   int &sp) {
    if constexpr (!MULTI) {
        return work_item(a, c, h, qt, sp);
    } else {
        const int lin = blockIdx.x;
        const int w = (lin % kXcds) * a.per_xcd + lin / kXcds;
        if (lin / kXcds >= a.per_xcd || w >= a.H * t.per_head) return false;
        h = w / t.per_head;
        int r = w % t.per_head, e = 0;
        while (e + 1 < t.n && r >= t.s[e].n_qtiles) {
            r -= t.s[e].n_qtiles;
            ++e;
        }
        qt = r;
        c = 0;
        sp = 0;
        const SubLaunch u = t.s[e];
        a.q_off = u.q_off; a.N_q = u.N_q; a.n_qtiles = u.n_qtiles;
        a.N_kv = u.N_kv; a.kv_start = u.kv_start; a.part_slot = u.part_slot;
        a.gap_row = u.gap_row; a.gap_len = u.gap_len;
        a.K += (size_t)u.kv_off * row_bytes;
        a.V += (size_t)u.kv_off * row_bytes;
        return true;
    }
}

// ------------------------------------------------------------------------------------------
// fp32: every operand as the sum of two fp16 numbers, multiplied on v_mfma_f32_32x32x16_f16.
//
// x = x1 + x2 with x1 = fp16(x), x2 = fp16(x - x1) is off by at most 2^-23 of x, and a product of two such sums is taken without x2*y2, which is
// at most 2^-22 of it: three matrix instructions of 32 cycles do what eight fp32 ones of 64 do, and their sums are rounded less often.  On N(0, 1)
// inputs results are 2.0e-7 to 3.6e-7 from fp64 (2-norm), with fp32 instructions they were 3.8e-7 to 7.1e-7.  (A logit that is one product alone, where
// roundings do not average, may be off by 2^-21 of itself; 2^-24 with fp32 instructions.)
// fp16's range is met by powers of two: one per query, one for the keys and one per feature of the values, from the first tile's
// largest numbers, which leaves a factor of 32 for those that follow.  Scaled numbers below 1/4 are off by half of the second part's step, 2^-25,
// whatever their size, so a workgroup keeps its result only if that is small beside it:
//   logits      what takes them from their sums to log2 units is within 2^-15.  Half a step of each of 128 numbers of a key, times a query's (below 2^15), then
//               makes 2^-18 of a logit at most and about a twentieth of that as such errors fall; half steps of a query's as much, twice with the largest keys.
//   by query    the largest |O| of the features is 2^20 times half a step of every value, and at least 2^-12 (beyond 128 keys: 2^-19 a key) of the largest
//               value: weights, whose half steps are 2^-36 of the largest one, then lose no more than fp32 sums do.
//   by feature  the same over four queries, with 2^18 and 2^-14, for features that have four adjacent keys whose values are below 2^-11 of the
//               first tile's (fewer, at the end: 2^-20) and not all 0.
// Otherwise, and with numbers beyond the factor of 32 or infinities, it does its work once more with v_mfma_f32_32x32x2_f32 on the
// numbers themselves, before any step if the first tile is enough to know.  tests/test_attention_f32_parts_bounds.py has this arithmetic for the CPU: what is kept is
// as good as plain fp32.  (Without the conditions one key at -1e9, a stand-in for -inf, in a window's first tile took the others' logits with it: O was
// off by 9e-3, at -1e12 by 0.8.)
//
// Four waves of 32 queries per workgroup, 32-key tiles, KG tiles at a time by as many groups of waves; KG == 1 leaves room for two
// workgroups on a compute unit, whose phases then overlap by themselves.  KG == 2: the groups' (O, max, sum) meet in
// LDS at the end, for small grids, whose key ranges would otherwise be many and their partial results with them.
// Tiles come to LDS as they are (global_load_lds), a step ahead.  The threads split each once for all waves, beside the matrix
// instructions of the phase before the one that reads it, and leave the parts in the order in which those are read:
//   K part p: [chunk of 8 features][key], V part p: [keys of a k slot group][feature] x 8 keys, 16 bytes each.
// Even features of V come first: a thread holds two adjacent ones and stores them apart.
//
// Bound by the matrix and the vector pipe together: a tile is 48 products (1,536 cycles) and about 300 vector instructions a wave, of which
// a third hides.  4 heads x 880 queries x 2,640 keys 64.5 -> 35.4 us (with its merge), 8 x 1,560 x 4,680 293 -> 126, 40 x 1,560 x 4,680 1,411 -> 565 (265 TFLOP/s), 1 x 128 x
// 30,000 248 -> 98, 6 x 250 x 100 25.0 -> 14.9.  (Three bf16 parts and six products: 50, 202, 897 us; its splitting in a phase of its own
// instead of beside the products: the same, as long as the compiler waited for the loads to LDS in front of every read of LDS, see load_to_lds.)
// ------------------------------------------------------------------------------------------
constexpr int kF32Waves = 4;                           // across the queries
constexpr int kF32Keys = 32;
constexpr int kF32Part = kF32Keys * 256;               // bytes of one part of a K or V tile
constexpr int kF32V = 2 * kF32Part;                    // K parts, V parts, K and V as they came
constexpr int kF32RawK = 4 * kF32Part;
constexpr int kF32RawV = kF32RawK + kF32Keys * 512;
constexpr int kF32Group = kF32RawV + kF32Keys * 512;   // LDS of a group of waves
constexpr int kF32Shared = 3 * 512 + 16;               // for all groups: see `shared` in the kernel
constexpr int kF32Lds = kF32Group + kF32Shared;
constexpr int kF32LdsPair = 2 * kF32Group + kF32Shared;
constexpr float kF32P = 0x1p11f;                       // what weights are scaled by
constexpr float kF32Zeros = 0x1p5f;                    // what keys and values are scaled by behind a first tile of zeros

#define WK_LDS(p) ((__attribute__((address_space(3))) void *)(p))
// typed LDS pointer from a 32-bit LDS byte address
#define WK_LDS_AT(T, addr) ((__attribute__((address_space(3))) T *)(size_t)(addr))
#define WK_GLB(p) ((const __attribute__((address_space(1))) void *)(p))

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// max over lanes l and l^32
__device__ inline float max_across_halves(float x) {
    const unsigned u = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// max over four adjacent lanes
__device__ inline float quad_max(float x) {
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xb1, 0xf, 0xf, false)));   // quad_perm [1, 0, 3, 2], [2, 3, 0, 1]
    return fmaxf(x, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x4e, 0xf, 0xf, false)));
}

__device__ inline float sum_across_halves(float x) {
    const unsigned u = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// max over a row of 16 lanes
__device__ inline float row_max(float x) {
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x128, 0xf, 0xf, false)));   // row_ror:8, 4, 2, 1
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x124, 0xf, 0xf, false)));
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x122, 0xf, 0xf, false)));
    return fmaxf(x, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x121, 0xf, 0xf, false)));
}

// 16 bytes per lane from base + offset to LDS, at `to` and on.  In assembly: the compiler waits for every load to LDS that it knows of in front of
// every read of LDS.  Its readers are behind a wait for all loads and a barrier; there is no output register to be waited for.
__device__ inline void load_to_lds(const char *base, unsigned offset, unsigned to) {
    unsigned callers_m0;   // m0 is the compiler's to manage: handed back as it was
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b32 m0, %0"
                 : "=&s"(callers_m0) : "s"(to), "v"(offset), "s"(base) : "memory");
}

// the two fp16 parts of two numbers times `up`, packed
struct Parts2 { unsigned p[2]; };
__device__ inline Parts2 split2(float x, float y, float up) {
    const f16x2 first = __builtin_convertvector(f32x2{x * up, y * up}, f16x2);
    const f16x2 second = {(_Float16)fmaf(x, up, -(float)first[0]), (_Float16)fmaf(y, up, -(float)first[1])};
    return Parts2{{__builtin_bit_cast(unsigned, first), __builtin_bit_cast(unsigned, second)}};
}

// The power of two that takes numbers up to `largest` below 2^(top + 1), of_zeros if all are 0; bad: there is none within 2^-60 .. 2^60 (infinities among others)
__device__ inline float scale_to(float largest, int top, float of_zeros, bool &bad) {
    const int e = (int)(__float_as_uint(largest) >> 23) & 0xff;
    if (largest == 0.f) return of_zeros;
    bad |= e < 127 + top - 60 || e > 127 + top + 60 || e > 127 + 50;
    return __uint_as_float((unsigned)min(max(254 + top - e, 1), 254) << 23);
}

__device__ inline float inverse(float power_of_two) { return __uint_as_float((254u << 23) - __float_as_uint(power_of_two)); }

// The A operands of the products, which come from LDS: read(p, t) is part p of fragment t.  A part is requested once its registers
// have been read by the fragment before, the first part, which is used last and longest, a fragment ahead.  The small
// products are added to `small`, which may be `c` itself: they come first.
template <typename Read>
struct PartStream {
    Read read;
    f16x8 first[2], second;
    __device__ inline PartStream(Read r) : read(r) {
        second = read(1, 0);
        first[0] = read(0, 0);
    }
    template <int N, typename Work>   // of N fragments; work(): other instructions beside the matrix ones
    __device__ inline void multiply(int t, const f16x8 (&y)[2], f32x16 &c, f32x16 &small, Work work) {
        __builtin_amdgcn_sched_barrier(0);
        if (t + 1 < N) first[(t + 1) & 1] = read(0, t + 1);
        small = __builtin_amdgcn_mfma_f32_32x32x16_f16(second, y[0], small, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (t + 1 < N) second = read(1, t + 1);
        work();
        small = __builtin_amdgcn_mfma_f32_32x32x16_f16(first[t & 1], y[1], small, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x16_f16(first[t & 1], y[0], c, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
};

template <int KG, bool MULTI, bool WITH_O>   // WITH_O: false: log-sum-exp only, V is not read
__global__ __launch_bounds__(KG * kF32Waves * 64, 2) void k_attn_f32(AttnArgs a, SubTable sub) {
    extern __shared__ __attribute__((aligned(256))) char smem[];
    int c, h, qt, sp;
    if (!select_work<MULTI>(a, sub, 512, c, h, qt, sp)) return;
    const Window win = window_of(a, c);
    const int n_kv = win.n_kv;
    float *const lse = win.lse;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qw = wave & 3, kg = KG == 1 ? 0 : wave >> 2;   // 32 queries of the workgroup's, tile of a step
    const int col = lane & 31, g = lane >> 5;
    const int q = qt * (kF32Waves * 32) + qw * 32 + col;
    const bool q_ok = q < a.N_q;
    const int q_ld = q_ok ? q : max(2 * a.N_q - 2 - q, 0);   // behind the last query the ones before it, so that a wave has few queries twice
    auto query_row = [&]() __attribute__((always_inline)) {
        int at = q_ld;
        asm("" : "+v"(at));
        return reinterpret_cast<const float *>(a.Q) + ((size_t)h * a.q_rows + a.q_off + at) * WK_D;
    };
    const bool partial_out = a.part_slot >= 0 || a.splits > 1;
    // this workgroup's keys [kt0, kt1): the whole window, or split sp of a.splits (whole tiles each)
    const int n_tiles = (n_kv + kF32Keys - 1) / kF32Keys;
    const int tiles_per_split = (n_tiles + a.splits - 1) / a.splits;
    const int kt0 = sp * tiles_per_split * kF32Keys;
    const int kt1 = min(n_kv, (sp + 1) * tiles_per_split * kF32Keys);

    if (kt0 >= kt1) {   // empty window, or a split past its end: contributes nothing
        if (kg > 0 || !q_ok) return;
        const size_t qrow = (size_t)h * a.q_rows + a.q_off + q, prow = (size_t)(a.part_slot >= 0 ? a.part_slot : sp) * a.H * a.q_rows + qrow;
        if (WITH_O) {
            float *out = partial_out ? a.part_o + prow * WK_D : reinterpret_cast<float *>(a.O) + qrow * WK_D;
            for (int c = g * 64; c < g * 64 + 64; c += 4) *reinterpret_cast<float4 *>(out + c) = float4{0, 0, 0, 0};
        }
        if (partial_out && g == 0) {
            a.part_ml[prow * 2] = -INFINITY;
            a.part_ml[prow * 2 + 1] = 0.f;
        }
        if (!partial_out && lse && g == 0) lse[qrow] = -INFINITY;
        return;
    }
    const bool idle = qt * (kF32Waves * 32) + qw * 32 >= a.N_q;   // no valid query in this wave: its loads, splits and barriers only

    const char *Kh = win.K + (size_t)h * win.stride * 512;
    const char *Vh = a.V + (size_t)h * win.stride * 512;
    char *const group = smem + kg * kF32Group;
    const unsigned lds0 = (unsigned)(size_t)WK_LDS(group);
    // shared: the first tiles' largest value of every feature, what takes its sums back, the largest of all its values as they are split; the first tiles' largest
    // key, whether the parts do not hold what they have to, whether a feature's values are of unlike size (sizes as int: their bits order as they do)
    int *const v_max = reinterpret_cast<int *>(smem + KG * kF32Group);
    float *const v_down = reinterpret_cast<float *>(v_max + WK_D);
    int *const v_seen = v_max + 2 * WK_D, *const k_max = v_max + 3 * WK_D, *const out_of_range = k_max + 1, *const mixed = k_max + 2;
    // Loads: wave qw fills two rows per load, of K rows 8*qw .. 8*qw+7, 16-byte chunk c of row k at slot c ^ (k & 15); of V the eight
    // rows 16*(qw/2) + 4*(qw%2) + {0..3, 8..11}, which a lane group multiplies at once, for the wave itself.
    // Rows past the range clamp to its last one (those keys are masked, their values cleared).
    // (addresses from a scalar base and a lane's 32-bit offset, made where they are used: kept, they would take 20 registers)
    const int v_key = 16 * (qw >> 1) + 4 * (qw & 1);
    auto issue_k = [&](int kt, unsigned place = kF32RawK) __attribute__((always_inline)) {
        size_t at = (size_t)kt * 512;
        unsigned l = lane;
        asm("" : "+s"(at), "+v"(l));
        const unsigned row = 8 * qw + (l >> 5), slot = ((l & 31) ^ (row & 15)) << 4, last = kt1 - 1 - kt;   // the range's last row, from the tile's first on
#pragma unroll
        for (unsigned i = 0; i < 4; ++i)
            load_to_lds(Kh + at, (min(row | 2 * i, last) << 9) | (slot ^ (i << 5)), lds0 + place + qw * 4096 + i * 1024);
    };
    auto issue_v = [&](int kt, unsigned place = kF32RawV) __attribute__((always_inline)) {
        size_t at = (size_t)kt * 512;
        unsigned l = lane;
        asm("" : "+s"(at), "+v"(l));
        const unsigned row = v_key + (l >> 5), last = kt1 - 1 - kt;
#pragma unroll
        for (unsigned e = 0; e < 8; e += 2)
            load_to_lds(Vh + at, (min(row + 8 * (e >> 2) + (e & 3), last) << 9) | ((l & 31) << 4), lds0 + place + qw * 4096 + e * 512);
    };
    // Queries come through LDS, the first and the second 64 features one after the other, in the wave's share of the parts' place: rows of 512 bytes, one
    // per lane, keep the L1 busy three times as long.  16-byte chunk c of row r at slot c ^ (r & 15).
    char *const q_lds = group + qw * (4 * kF32Part / kF32Waves);
    auto issue_q = [&](unsigned half) __attribute__((always_inline)) {
        unsigned l = lane;
        asm("" : "+v"(l));
        const int q0 = qt * (kF32Waves * 32) + qw * 32, first = max(q0 - 32, 0), last = a.N_q - 1 - first;   // (rows from `first` on)
        const char *base = a.Q + ((size_t)h * a.q_rows + a.q_off + first) * 512;
#pragma unroll
        for (unsigned i = 0; i < 8; ++i) {
            const unsigned row = 4 * i + (l >> 4);
            const int at = q0 - first + (int)row;
            load_to_lds(base, ((unsigned)max(min(at, 2 * last - at), 0) << 9) | (half << 8) | (((l & 15) ^ (row & 15)) << 4), lds0 + qw * (4 * kF32Part / kF32Waves) + i * 1024);
        }
    };
    if (!idle) issue_q(0);
    const bool any = kt0 + kg * kF32Keys < kt1;   // with a single tile the second group has none
    if (any) {
        issue_k(kt0 + kg * kF32Keys);
        if (WITH_O) issue_v(kt0 + kg * kF32Keys);
    }
    for (int i = tid; i < kF32Shared / 4; i += KG * kF32Waves * 64) v_max[i] = 0;

    // B operand of S^T = K Q^T: k slot 8*g + e of step s means feature 16*s + 8*g + e
    f16x8 qr[8][2];
    bool bad_keys = false;   // or queries
    float to_log2 = a.scale_log2;   // of this lane's query: what takes scores as they are summed to log2 units
    if (!idle) {
        float4 x[16];
        auto read_q = [&](int half) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                x[8 * half + i] = *reinterpret_cast<const float4 *>(q_lds + col * 256 + (((4 * (i >> 1) + 2 * g + (i & 1)) ^ (col & 15)) << 4));
        };
        if (any) __builtin_amdgcn_s_waitcnt(WITH_O ? 0x0F78 : 0x0F74);   // all but the keys' and values' loads, four each
        else __builtin_amdgcn_s_waitcnt(0x0F70);
        asm volatile("" ::: "memory");
        read_q(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // before the place is written again
        issue_q(1);
        __builtin_amdgcn_s_waitcnt(0x0F70);
        asm volatile("" ::: "memory");
        read_q(1);
        float largest = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i)
            largest = fmaxf(fmaxf(fmaxf(largest, fabsf(x[i].x)), fabsf(x[i].y)), fmaxf(fabsf(x[i].z), fabsf(x[i].w)));
        const float up = scale_to(max_across_halves(largest), 14, 0x1p40f, bad_keys);   // (zeros have all the range)
        to_log2 *= inverse(up);
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            Parts2 t[4];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const float4 y = x[2 * s + u];
                t[2 * u] = split2(y.x, y.y, up);
                t[2 * u + 1] = split2(y.z, y.w, up);
            }
#pragma unroll
            for (int p = 0; p < 2; ++p) qr[s][p] = __builtin_bit_cast(f16x8, u32x4{t[0].p[p], t[1].p[p], t[2].p[p], t[3].p[p]});
        }
    }
    f32x16 o[4];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[b][r] = 0.f;
    // (finite: scores of -inf then have weight 0 also in tiles that hold nothing else, whichever wave group or key range
    // begins with one)
    float m_run = -FLT_MAX, l_run = 0.f;

    // scores of the keys from kt on to their weights; accumulator register r of this lane is key kt + 8*(r/4) + 4*g + r%4
    auto softmax = [&](f32x16 &s, int kt) __attribute__((always_inline)) {
        if (kt + kF32Keys > kt1) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (kt + 8 * (r >> 2) + 4 * g + (r & 3) >= kt1) s[r] = -INFINITY;
        }
        float m_tile = s[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) m_tile = fmaxf(m_tile, s[r]);
        m_tile = max_across_halves(m_tile) * to_log2;
        if (__any(m_tile > m_run + 4.f)) {   // the maximum moves where weights would grow beyond 2^4, 2^15 as they are split
            const float m_new = fmaxf(m_run, m_tile), alpha = __builtin_amdgcn_exp2f(m_run - m_new);
            l_run *= alpha;
            m_run = m_new;
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[b][r] *= alpha;
        }
        float l_tile[4];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], to_log2, -m_run));
            l_tile[r & 3] = r < 4 ? s[r] : l_tile[r & 3] + s[r];
        }
        l_run += (l_tile[0] + l_tile[1]) + (l_tile[2] + l_tile[3]);
    };

    // A thread's share of a tile, in quarters: four numbers of K (of a row) or of V (of four keys) are read, and split and left a call later
    float quarter[4], k_largest = 0.f, v_largest[2] = {0.f, 0.f};   // (of all tiles)
    unsigned v_least[2] = {~0u, ~0u};   // the smallest of the four keys' largest, as bits less 1, so that it is none that is all zeros
    float k_up = 1.f, v_up[2] = {1.f, 1.f};
    int me = tid;
    auto k_from = [&](int c) __attribute__((always_inline)) {   // features 8 * ((me >> 5 & 7) + 8 * (c / 2)) + 4 * (c % 2) of key me % 32
        const int chunk = 2 * ((me >> 5) & 7) + 16 * (c >> 1) + (c & 1);
        return *reinterpret_cast<const float4 *>(group + kF32RawK + (me & 31) * 512 + ((chunk ^ (me & 15)) << 4));
    };
    auto v_from = [&](int f, int e) __attribute__((always_inline)) {   // feature 2 * lane + f of the wave's row e
        return *reinterpret_cast<const float *>(group + kF32RawV + (qw * 8 + e) * 512 + (me & 63) * 8 + f * 4);
    };
    auto quarter_top = [&]() __attribute__((always_inline)) {
        return fmaxf(fmaxf(fmaxf(fabsf(quarter[0]), fabsf(quarter[1])), fabsf(quarter[2])), fabsf(quarter[3]));
    };
    auto store_quarter = [&](char *to, float up) __attribute__((always_inline)) {
        const Parts2 x = split2(quarter[0], quarter[1], up), y = split2(quarter[2], quarter[3], up);
#pragma unroll
        for (int p = 0; p < 2; ++p) *reinterpret_cast<uint2 *>(to + p * kF32Part) = uint2{x.p[p], y.p[p]};
    };
    auto k_work = [&](int t) __attribute__((always_inline)) {
        const int c = t >> 1;
        if ((t & 1) == 0) {
            const float4 x = k_from(c);
            quarter[0] = x.x; quarter[1] = x.y; quarter[2] = x.z; quarter[3] = x.w;
        } else {
            k_largest = fmaxf(k_largest, quarter_top());
            store_quarter(group + (((me >> 5) & 7) + 8 * (c >> 1)) * 512 + (me & 31) * 16 + (c & 1) * 8, k_up);
        }
    };
    auto v_work = [&](int t, int kt) __attribute__((always_inline)) {
        const int f = t >> 2, half = (t >> 1) & 1;
        if ((t & 1) == 0) {
#pragma unroll
            for (int u = 0; u < 4; ++u) quarter[u] = v_from(f, 4 * half + u);
        } else {
            if (kt + kF32Keys > kt1)   // rows past the range: the last one may be infinite
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (kt + v_key + 8 * half + u >= kt1) quarter[u] = 0.f;
            float top = quarter_top();
            v_largest[f] = fmaxf(v_largest[f], top);
            if (kt + v_key + 8 * half + 4 > kt1) top *= 0x1p9f;   // (less than four keys: now and then all small in some feature)
            v_least[f] = min(v_least[f], __float_as_uint(top) - 1);
            store_quarter(group + kF32V + qw * 2048 + f * 1024 + (me & 63) * 16 + half * 8, v_up[f]);
        }
    };
    auto begin_share = [&]() __attribute__((always_inline)) {
        me = tid;
        asm("" : "+v"(me));   // (its addresses are not kept either)
    };
    constexpr float kLimit = 65504.f;   // fp16's largest number

    // the scales, from the first tiles
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wave's part of the first tile has landed
    __syncthreads();
    if (any) {
        float top = 0.f;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float4 x = k_from(c);
            top = fmaxf(fmaxf(fmaxf(top, fabsf(x.x)), fabsf(x.y)), fmaxf(fabsf(x.z), fabsf(x.w)));
        }
        top = row_max(top);
        if ((lane & 15) == 0) atomicMax(k_max, __float_as_int(top));
        if (WITH_O)
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                top = 0.f;
#pragma unroll
                for (int e = 0; e < 8; ++e) top = fmaxf(top, fabsf(v_from(f, e)));
                atomicMax(v_max + 2 * lane + f, __float_as_int(top));
            }
    }
    __syncthreads();
    bool bad_values = false;
    k_up = scale_to(__int_as_float(*k_max), 10, kF32Zeros, bad_keys);
    to_log2 *= inverse(k_up);
    if (WITH_O)
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            v_up[f] = scale_to(__int_as_float(v_max[2 * lane + f]), 10, kF32Zeros, bad_values);
            if (wave == 0) v_down[2 * lane + f] = inverse(kF32P * v_up[f]);
        }
    if (any)
#pragma unroll
        for (int t = 0; t < 8; ++t) k_work(t);
    if (bad_keys || bad_values || (!idle && to_log2 > 0x1p-15f)) *out_of_range = 1;

    // The steps.  Beside the products of S^T a wave splits its share of the tile's values, beside those of O^T its share of the next tile's
    // keys (without a next tile: of the last one's again, which nothing reads)
    auto meet_keys = [&]() __attribute__((always_inline)) {   // K's parts are there, the values before are consumed
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wave's values have landed
        __syncthreads();
    };
    auto meet_values = [&]() __attribute__((always_inline)) {   // V's parts are there, K's are consumed
        __builtin_amdgcn_s_waitcnt(WITH_O ? 0x0F74 : 0x0F70);   // this wave's keys of the next tile have landed; its values, four loads, are behind them
        __syncthreads();
    };
    meet_keys();
    const bool steps = __builtin_amdgcn_readfirstlane(*out_of_range) == 0;   // (not behind a first tile that leads to fp32 products as it is)
    const int n_steps = steps ? ((kt1 - kt0 + kF32Keys - 1) / kF32Keys + KG - 1) / KG : 0;
    const int my_steps = steps ? (kt1 - kt0 - kg * kF32Keys + KG * kF32Keys - 1) / (KG * kF32Keys) : 0;   // with an odd count of tiles the second group has one less
    int kt = kt0 + kg * kF32Keys;
    constexpr int kStep = KG * kF32Keys;
    if (KG == 2 && kg == 0) __builtin_amdgcn_s_setprio(1);   // one of a SIMD's two waves ahead: one does its softmax while the other multiplies
    if (!idle) {
        for (int j = 0; j < my_steps; ++j, kt += kStep) {
            if (j > 0) meet_keys();
            if (kt + kStep < kt1) issue_k(kt + kStep);
            begin_share();
            f32x16 s, small;   // (apart: eight roundings at the size of a score instead of 24)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = small[r] = 0.f;
            const unsigned k_at = lds0 + ((me >> 5) & 1) * 512 + (me & 31) * 16;
            PartStream k([&](int p, int t) __attribute__((always_inline)) { return *WK_LDS_AT(const f16x8, k_at + p * kF32Part + t * 1024); });
#pragma unroll
            for (int t = 0; t < 8; ++t)
                k.template multiply<8>(t, qr[t], s, small, [&]() __attribute__((always_inline)) {
                    if (WITH_O) v_work(t, kt);
                });
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] += small[r];
            if (WITH_O && kt + kStep < kt1) issue_v(kt + kStep);   // (the wave's own rows: no other reads them)
            softmax(s, kt);
            f16x8 pr[2][2];
            if (WITH_O)
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    Parts2 u[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) u[e] = split2(s[8 * t + 2 * e], s[8 * t + 2 * e + 1], kF32P);
#pragma unroll
                    for (int p = 0; p < 2; ++p) pr[t][p] = __builtin_bit_cast(f16x8, u32x4{u[0].p[p], u[1].p[p], u[2].p[p], u[3].p[p]});
                }
            meet_values();
            begin_share();
            if (WITH_O) {
                // O^T += V^T P^T: k slot 8*g + e of step t means key 16*t + 8*(e/4) + 4*g + e%4, accumulator register 8*t + e;
                // row i of block b is feature 2*(32*(b%2) + i) + b/2
                const unsigned v_at = lds0 + kF32V + ((me >> 5) & 1) * 2048 + (me & 31) * 16;
                PartStream v([&](int p, int i) __attribute__((always_inline)) {   // i = 2*b + t
                    return *WK_LDS_AT(const f16x8, v_at + p * kF32Part + (i & 1) * 4096 + (i >> 1) * 512);
                });
#pragma unroll
                for (int b = 0; b < 4; ++b) {   // sums of the tile's products by themselves: one rounding at the size of O per tile, not six, for 4 % of the time
                    f32x16 sum;
#pragma unroll
                    for (int r = 0; r < 16; ++r) sum[r] = 0.f;
                    v.template multiply<8>(2 * b, pr[0], sum, sum, [&]() __attribute__((always_inline)) { k_work(2 * b); });
                    v.template multiply<8>(2 * b + 1, pr[1], sum, sum, [&]() __attribute__((always_inline)) { k_work(2 * b + 1); });
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[b][r] += sum[r];
                    asm volatile("" : "+v"(o[b]));   // (here: put off, four sums would be held)
                }
            } else {
#pragma unroll
                for (int t = 0; t < 8; ++t) k_work(t);
            }
        }
    } else {
        for (int j = 0; j < my_steps; ++j, kt += kStep) {
            if (j > 0) meet_keys();
            if (kt + kStep < kt1) issue_k(kt + kStep);
            begin_share();
            if (WITH_O)
#pragma unroll
                for (int t = 0; t < 8; ++t) v_work(t, kt);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // before the place is written again
            if (WITH_O && kt + kStep < kt1) issue_v(kt + kStep);
            meet_values();
            begin_share();
#pragma unroll
            for (int t = 0; t < 8; ++t) k_work(t);
        }
    }
    if (my_steps < n_steps) {   // the other group's last tile
        begin_share();
        if (my_steps > 0) meet_keys();
        meet_values();
    }
    // What was met, and whether the parts lose too much by it, see above.
    bool lost = k_largest * k_up >= kLimit;
    if (WITH_O)
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            v_largest[f] *= v_up[f];
            atomicMax(v_seen + 2 * lane + f, __float_as_int(v_largest[f]));
            lost |= v_largest[f] >= kLimit;
            if (v_least[f] != ~0u && __uint_as_float(v_least[f] + 1) * v_up[f] < 0.5f) v_max[2 * lane + f] = *mixed = -1;   // (no longer needed as it was)
        }
    if (!WITH_O && lost) *out_of_range = 1;
    __syncthreads();   // every wave is done with its last tile, and its share of the LDS free
    if (WITH_O && my_steps > 0 && !idle) {
        const float l_tot = sum_across_halves(l_run);
        float of_values = 0.f, of_weights = 0.f;   // the features' largest, of a lane's two at first
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            const float seen = __int_as_float(v_seen[2 * lane + f]), down = v_down[2 * lane + f];
            of_weights = fmaxf(of_weights, seen * down);
            of_values = fmaxf(of_values, seen > 0.f ? down : 0.f);
        }
        of_weights = row_max(of_weights);
        of_values = row_max(of_values);
        of_weights = max_across_halves(fmaxf(of_weights, __shfl_xor(of_weights, 16)));
        of_values = max_across_halves(fmaxf(of_values, __shfl_xor(of_values, 16)));
        const float least = fmaxf(of_weights * kF32P * fmaxf(0x1p-12f, (float)(my_steps * kF32Keys) * 0x1p-19f), of_values * 64.f * l_tot);
        // by 16-byte chunks of features, as they are stored below: read(chunk), then use(its feature i, that one's register: block and number)
        auto each = [&](auto read, auto use) __attribute__((always_inline)) {
#pragma unroll
            for (int n = 0; n < 16; ++n) {
                const int b = n >> 3, t = (n >> 1) & 3, u = 2 * (n & 1), chunk = 16 * b + 4 * t + 2 * g + u / 2;
                read(chunk);
#pragma unroll
                for (int i = 0; i < 4; ++i) use(i, b + 2 * (i & 1), 4 * t + u + (i >> 1));
            }
        };
        if (__builtin_amdgcn_readfirstlane(*mixed) != 0) {
            int4 of_unlike_size;
            float4 seen;
            each([&](int chunk) __attribute__((always_inline)) {
                of_unlike_size = *reinterpret_cast<const int4 *>(v_max + 4 * chunk);
                seen = *reinterpret_cast<const float4 *>(v_seen + 4 * chunk);
            }, [&](int i, int b, int r) __attribute__((always_inline)) {
                const float at_least = fmaxf((&seen.x)[i] * (kF32P * 0x1p-14f), 16.f * l_tot);
                lost |= quad_max(fabsf(o[b][r])) < ((&of_unlike_size.x)[i] < 0 ? at_least : 0.f);
            });
        }
        float4 down;
        float row = 0.f;
        each([&](int chunk) __attribute__((always_inline)) { down = *reinterpret_cast<const float4 *>(v_down + 4 * chunk); },
             [&](int i, int b, int r) __attribute__((always_inline)) {
                 o[b][r] *= (&down.x)[i];
                 row = fmaxf(row, fabsf(o[b][r]));
             });
        lost |= max_across_halves(row) < least;
    }
    if constexpr (WITH_O) {
        if (lost) *out_of_range = 1;
        __syncthreads();
    }
    // (looked at here only: behind every barrier, and with the values requested behind the second one, 4 heads x 880 queries x 2,640 keys in one
    // range took 129 us, now 125)
    const bool exact = __builtin_amdgcn_readfirstlane(*out_of_range) != 0;
    // Once more from the first tile on, with fp32 operands: tiles as they come, in the raw tiles' place and in the parts' in turn.  Bound by the products, 128 of 64 cycles a tile.  With
    // a key at -inf in the first tile, which is known before any step, 4 heads x 880 queries x 2,640 keys take 72 us, 8 x 1,560 x 4,680 216, 1 x 128 x 30,000 254 (operands
    // straight from memory and behind all the steps: 96, 388, 380; the kernel of fp32 products alone, for any keys, 64, 295, 252); found out at the end
    // only, by the values' spread, 93, 418 and 338.
    if (exact) {
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[b][r] = 0.f;
        m_run = -FLT_MAX;
        l_run = 0.f;
        to_log2 = 1.f;   // (rounded before the maximum is taken: a fused product would differ from it by 2^-24 of itself, beyond 2^31 by more than exp2 can hold)
        float4 y[16];
        if (!idle) {
            const float *Qrow = query_row();
#pragma unroll
            for (int t = 0; t < 16; ++t) y[t] = *reinterpret_cast<const float4 *>(Qrow + 8 * t + 4 * g);
        }
        const int all_steps = ((kt1 - kt0 + kF32Keys - 1) / kF32Keys + KG - 1) / KG;
        int kt = kt0 + kg * kF32Keys;
        if (kt < kt1) {
            issue_k(kt);
            if (WITH_O) issue_v(kt);
        }
        for (int j = 0; j < all_steps; ++j, kt += kStep) {
            const unsigned place = j & 1 ? 0u : kF32RawK, next = kF32RawK - place;
            __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wave's share has landed
            asm volatile("" ::: "memory");
            if (WITH_O && kt < kt1 && kt + kF32Keys > kt1) {   // values past the range become zeros: the last row there may be infinite
#pragma unroll
                for (int e = 0; e < 8; e += 2)
                    if (kt + v_key + 8 * (e >> 2) + (e & 3) + (lane >> 5) >= kt1)
                        *reinterpret_cast<float4 *>(group + place + kF32Keys * 512 + qw * 4096 + e * 512 + lane * 16) = float4{0, 0, 0, 0};
            }
            __syncthreads();   // everyone's has, and the tile before is consumed
            if (kt + kStep < kt1) {
                issue_k(kt + kStep, next);
                if (WITH_O) issue_v(kt + kStep, next + kF32Keys * 512);
            }
            if (kt >= kt1 || idle) continue;
            // operands are read two groups of four products ahead, and the order is kept
            unsigned at = lds0 + place;
            asm("" : "+s"(at));
            f32x4 ka[3];
            f32x2 va[3][2];   // of features 64 * b + 2 * col and one more, of which the second's block is b + 2
            auto read_k = [&](int t) __attribute__((always_inline)) { ka[t % 3] = *WK_LDS_AT(const f32x4, at + col * 512 + (((2 * t + g) ^ (col & 15)) << 4)); };
            auto read_v = [&](int r) __attribute__((always_inline)) {
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    va[r % 3][b] = *WK_LDS_AT(const f32x2, at + kF32Keys * 512 + ((2 * (r >> 3) + g) * 8 + 4 * ((r >> 2) & 1) + (r & 3)) * 512 + b * 256 + col * 8);
            };
            f32x16 s;
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = 0.f;
            read_k(0);
            read_k(1);
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                if (t + 2 < 16) read_k(t + 2);
                else if (WITH_O) read_v(t - 14);
                __builtin_amdgcn_sched_barrier(0);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(ka[t % 3][0], y[t].x, s, 0, 0, 0);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(ka[t % 3][1], y[t].y, s, 0, 0, 0);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(ka[t % 3][2], y[t].z, s, 0, 0, 0);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(ka[t % 3][3], y[t].w, s, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] *= a.scale_log2;
            softmax(s, kt);
            if (!WITH_O) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                if (r + 2 < 16) read_v(r + 2);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int b = 0; b < 4; ++b) o[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[r % 3][b & 1][b >> 1], s[r], o[b], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();   // the last tiles are consumed
    }
    // The wave groups meet: waves 4..7 leave (O^T, max, sum) of their keys in LDS, waves 0..3 add them to theirs.
    // Register r of a wave's lane sits at [qw][r][lane]: consecutive lanes, consecutive banks.
    if constexpr (KG == 2) {
        float *meet = reinterpret_cast<float *>(smem) + qw * (66 * 64) + lane;
        if (kg == 1) {
            if (WITH_O)
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int r = 0; r < 16; ++r) meet[(16 * b + r) * 64] = o[b][r];
            meet[64 * 64] = m_run;
            meet[65 * 64] = l_run;
        }
        __syncthreads();
        if (kg == 1) return;
        const float m_other = meet[64 * 64];   // -FLT_MAX, with sums of 0, if the second group had no tile
        const float m_new = fmaxf(m_run, m_other);
        const float w0 = __builtin_amdgcn_exp2f(m_run - m_new), w1 = __builtin_amdgcn_exp2f(m_other - m_new);
        m_run = m_new;
        l_run = fmaf(w1, meet[65 * 64], w0 * l_run);
        if (WITH_O)
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[b][r] = fmaf(w1, meet[(16 * b + r) * 64], w0 * o[b][r]);
    }
    if (idle) return;
    int q_at = q_ld;
    asm("" : "+v"(q_at));   // (rows of the results from here on, not kept through the loop)
    const size_t qrow = (size_t)h * a.q_rows + a.q_off + q_at, prow = (size_t)(a.part_slot >= 0 ? a.part_slot : sp) * a.H * a.q_rows + qrow;
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    if (q_ok && !partial_out && lse && g == 0) lse[qrow] = (m_run + log2f(l_tot)) * 0.6931471805599453f;
    if (q_ok && partial_out && g == 0) {   // (O, max, sum) of this key range, merged by k_attn_merge
        a.part_ml[prow * 2] = m_run;
        a.part_ml[prow * 2 + 1] = l_tot;
    }
    if (!WITH_O) return;
    // O leaves through the wave's own LDS, so that a store has two whole rows, not 16 bytes of 32 (with the queries' way: 4 heads x 880
    // queries x 2,640 keys in 9 ranges 38.0 -> 36.4 us): chunk c of row r at slot
    // c ^ (r & 15)
    char *const o_lds = smem + qw * (KG == 2 ? 66 * 64 * 4 : 32 * 512);
    const float inv = partial_out ? 1.f : 1.f / l_tot;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int u = 0; u < 4; u += 2) {
                const int chunk = 16 * b + 4 * t + 2 * g + u / 2;
                *reinterpret_cast<float4 *>(o_lds + col * 512 + ((chunk ^ (col & 15)) << 4)) =
                    float4{o[b][4 * t + u] * inv, o[b + 2][4 * t + u] * inv, o[b][4 * t + u + 1] * inv, o[b + 2][4 * t + u + 1] * inv};
            }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    const int q0 = qt * (kF32Waves * 32) + qw * 32, rows = min(32, a.N_q - q0);
    const size_t row0 = (size_t)h * a.q_rows + a.q_off + q0;
    char *const out = partial_out ? reinterpret_cast<char *>(a.part_o) + ((size_t)(a.part_slot >= 0 ? a.part_slot : sp) * a.H * a.q_rows + row0) * 512
                                  : a.O + row0 * 512;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int row = 2 * i + (lane >> 5), chunk = lane & 31;
        if (row < rows) *reinterpret_cast<float4 *>(out + (size_t)row * 512 + chunk * 16) = *reinterpret_cast<const float4 *>(o_lds + row * 512 + ((chunk ^ (row & 15)) << 4));
    }
}

// ------------------------------------------------------------------------------------------
// bf16: v_mfma_f32_32x32x16_bf16, waves of 32 queries, 64-key tiles.
//
// QW == 8: 256 queries in eight waves, every wave multiplies every tile.  QW == 4, KG == 1: 128 queries in four waves, the same
// steps (compiled; the hand-scheduled loop is for eight waves), for small grids of short windows.  KG == 2 (grids that would leave compute units idle): 128
// queries; waves 0..3 take the even tiles and waves 4..7 the odd ones for the same queries, and their (O, max, sum) meet
// in LDS at the end.  That keeps two waves on every SIMD, so that one covers the other's waits: 12 heads x 2,640 queries x
// 10,560 keys take 162 us, against 178 us with workgroups of four waves (one per SIMD) and 229 us with QW == 8
// (132 workgroups for 256 compute units).  Splitting each tile's keys between the two wave groups instead, with one
// tile per step, halves the work between barriers: 177 us.
//
// K and V tiles go from global memory straight into a 4-deep LDS ring (global_load_lds, no
// register staging), K tiles four and V tiles three ahead of the step that loads them, which
// gives each three steps to land (S^T is formed one step early, so K leads V by one tile).  Both tiles are row-major with their
// 16-byte chunks permuted inside a row; the permutation is applied on the source side (each
// lane fetches the chunk that belongs in its linear LDS slot).  K^ operands are plain 16-byte
// reads; V^T operands are LDS transpose reads (ds_read_b64_tr_b16) of the row-major V tile.
// While a wave turns S^T of tile j into probabilities and multiplies them into O^T it already
// computes S^T of tile j+1, so the softmax arithmetic has independent matrix work to hide under.
// ------------------------------------------------------------------------------------------
constexpr int kKeys = 64;               // keys per tile
constexpr int kTileBytes = kKeys * 256; // one K or V tile
constexpr int kStages = 4;
constexpr int kVRing = kStages * kTileBytes;          // K ring at 0, V ring behind it
constexpr int kRings = 2 * kStages * kTileBytes;   // 128 KB
constexpr int kSmemBytes = kRings + 512 + 16;      // KG == 2: and the first tile's row maxima of 128 queries; whether the work is to be done once more

typedef short i16x4 __attribute__((ext_vector_type(4)));

__device__ inline float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

// registers the hand-scheduled loop uses beyond its operands: the odd-position S^T tile, P, the K and V^T
// fragment buffers and two temporaries
#define WK_ATTN_LOOP_CLOBBERS \
    "v96", "v97", "v98", "v99", "v100", "v101", "v102", "v103", "v104", "v105", "v106", "v107", \
    "v108", "v109", "v110", "v111", "v112", "v113", "v114", "v115", "v116", "v117", "v118", "v119", \
    "v120", "v121", "v122", "v123", "v124", "v125", "v126", "v127", "v160", "v161", "v162", "v163", \
    "v164", "v165", "v166", "v167", "v168", "v169", "v170", "v171", "v172", "v173", "v174", "v175", \
    "v176", "v177", "v178", "v179", "v180", "v181", "v182", "v183", "v184", "v185", "v186", "v187", \
    "v188", "v189", "v190", "v191", "v192", "v193", "v194", "v195", "v196", "v197", "v198", "v199", \
    "v200", "v201", "v202", "v203", "v204", "v205", "v206", "v207", "v208", "v209", "v210", "v211", \
    "v212", "v213", "v214", "v215", "v216", "v217", "v218", "v219", "v220", "v221", "v222", "v223", \
    "v244", "v245"

// IN_PLACE: the window is a list of segments (the native rows, then each retrieved chunk where the store
// keeps it) instead of one array.  Tiles never straddle segments: a segment's last tile may be partial and
// is masked like the window's last tile; a wave-uniform cursor walks the list.
constexpr int kMaxSegments = 33;   // native rows + up to 32 retrieved chunks
struct Segment { const char *K; const char *V; int len; int pad; };

using wk::uniform_ptr;

// One pass over a workgroup's keys.  QW: waves across the queries; KG: wave groups, which take alternate tiles; TRIPS: by the hand-scheduled loop
// where that can run.  It has no running maximum: where scores grow by more than fp32 can hold within a trip, or weights times values
// do, it leaves infinities or NaN; then true is returned in every thread, and stored says of each wave whether its results hold and are in place (a pass
// of that wave's stores nothing).
template <int QW, int KG, bool MULTI, bool IN_PLACE, bool GAP, bool TRIPS>
__device__ __attribute__((always_inline)) inline bool attend(AttnArgs a, const SubTable &sub, const int wave, bool &stored) {
    static_assert((QW == 8 && KG == 1) || (QW == 4 && (KG == 1 || KG == 2)), "one tile, or a pair of tiles, per step");
    constexpr int NB = 16 / (QW * KG); // 1 KB blocks of a tile that a wave loads
    // s_waitcnt vmcnt(4 * NB) alone: all but the last four tile shares have landed
    constexpr int kWaitTwoSteps = NB == 2 ? 0x0F78 : 0x4F70;
    constexpr int kWaitAll = 0x0F70;        // vmcnt(0)
    static_assert(!(MULTI && IN_PLACE), "a table of launches over one window array only");
    static_assert(MULTI || !GAP, "gaps belong to a table's entries");
    extern __shared__ __attribute__((aligned(256))) char smem[];
    int c, h, qt, sp;
    if (!select_work<MULTI>(a, sub, 256, c, h, qt, sp)) return false;
    const Window win = window_of(a, c);
    float *const lse = win.lse;
    int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0));
    asm volatile("" : "+v"(lane));   // (what one pass makes of it is not kept for another)
    const int tid = wave * 64 + lane;
    // segment list of this head and its number of tiles
    int n_seg = 0, seg_tiles = 0;
    const Segment *seg_list = nullptr;
    if constexpr (IN_PLACE) {
        __shared__ Segment segs[kMaxSegments];
        __shared__ Segment raw[kMaxSegments];
        __shared__ int seg_meta[2];
        // entry 0 = native rows, entry 1 + r = retrieved chunk r; one thread each fetches its entry (the
        // id, then the chunk's length and addresses), thread 0 then drops the empty ones
        if (tid <= a.R_max) {
            Segment e{nullptr, nullptr, 0, 0};
            if (tid == 0) {
                if (a.N_kv > 0)
                    e = Segment{a.K + (size_t)h * a.kv_row_stride * 256, a.V + (size_t)h * a.kv_row_stride * 256, a.N_kv, 0};
            } else {
                int nf = a.n_ids ? *a.n_ids : a.R_max;
                nf = nf < a.R_max ? nf : a.R_max;
                const int id = tid - 1 < nf ? a.ids[tid - 1] : -1;
                if (id >= 0 && id < a.store_M) {
                    const int len = a.n_tok[id];
                    if (len > 0 && len <= a.max_tok)   // a chunk beyond the descriptor's bound is skipped
                        e = Segment{reinterpret_cast<const char *>(a.k_table[id]) + (size_t)h * len * 256,
                                    reinterpret_cast<const char *>(a.v_table[id]) + (size_t)h * len * 256, len, 0};
                }
            }
            raw[tid] = e;
        }
        __syncthreads();
        if (tid == 0) {
            int n = 0, tiles = 0;
            for (int r = 0; r <= a.R_max; ++r) {
                const Segment e = raw[r];
                if (e.len > 0) {
                    segs[n++] = e;
                    tiles += (e.len + 63) / 64;
                }
            }
            seg_meta[0] = n;
            seg_meta[1] = tiles;
        }
        __syncthreads();
        n_seg = __builtin_amdgcn_readfirstlane(seg_meta[0]);
        seg_tiles = __builtin_amdgcn_readfirstlane(seg_meta[1]);
        seg_list = segs;
    }
    // IN_PLACE: only its tile count is used; GAP: the rows behind the gap move up to its start
    const int n_kv = IN_PLACE ? seg_tiles * 64 : GAP ? min(win.n_kv, max(a.gap_row, win.n_kv - a.gap_len)) : win.n_kv;
    const unsigned gap_from = (unsigned)a.gap_row * 256u, gap_bytes = (unsigned)a.gap_len * 256u;
    auto skip_gap = [&](unsigned off) { return GAP && off >= gap_from ? off + gap_bytes : off; };
    const int col = lane & 31, g = lane >> 5;
    const int qw = KG == 1 ? wave : wave & 3, kg = KG == 1 ? 0 : wave >> 2;   // 32 queries of the workgroup's, tile of every pair (KG == 2)
    const int q = qt * (QW * 32) + qw * 32 + col;
    const bool q_ok = q < a.N_q;
    const int q_ld = q_ok ? q : a.N_q - 1;
    const char *Qrow = a.Q + ((size_t)h * a.q_rows + a.q_off + q_ld) * 256;
    const bool partial_out = a.splits > 1 || a.part_slot >= 0;  // (O, max, sum) for k_attn_merge
    // rows of this lane's query in O / lse and in the partial arrays (formed where they are used:
    // two 64-bit values per lane are not worth carrying through the loop)
    auto out_row = [&]() { return (size_t)h * a.q_rows + a.q_off + q; };
    auto part_row = [&]() { return ((size_t)(a.part_slot >= 0 ? a.part_slot : sp) * a.H + h) * a.q_rows + a.q_off + q; };

    // this workgroup's tiles [t0, t1) of the window
    const int n_tiles = (n_kv + kKeys - 1) / kKeys;
    const int tiles_per_split = (n_tiles + a.splits - 1) / a.splits;
    const int t0 = sp * tiles_per_split;
    const int t1 = min(n_tiles, t0 + tiles_per_split);
    if (t0 >= t1) {   // empty window, or a split past its end: contributes nothing
        if (q_ok) {
            if (!partial_out) {
                const size_t qrow = out_row();
                char *Orow = a.O + qrow * 256;
                for (int c = g * 8; c < g * 8 + 8; ++c) reinterpret_cast<uint4 *>(Orow)[c] = uint4{0, 0, 0, 0};
                if (lse && g == 0) lse[qrow] = -INFINITY;
            } else {
                const size_t prow = part_row();
                for (int c = g * 16; c < g * 16 + 16; ++c) reinterpret_cast<float4 *>(a.part_o + prow * WK_D)[c] = float4{0, 0, 0, 0};
                if (g == 0) { a.part_ml[prow * 2] = -INFINITY; a.part_ml[prow * 2 + 1] = 0.f; }
            }
        }
        return false;
    }

    // B operand of S^T = K Q^T, step st: features 16*st + 8*g .. +7 of this lane's query
    bf16x8 qb[8];
#pragma unroll
    for (int st = 0; st < 8; ++st) qb[st] = *reinterpret_cast<const bf16x8 *>(Qrow + (2 * st + g) * 16);

    // K tile: row-major, chunk c of key k at slot c ^ (k & 15).  A operand of S^T block b, step st:
    // key 32*b + col, chunk 2*st + g.   address = k_rd[st] + stage*16384 + b*8192
    // (operand read addresses are kept as 32-bit LDS addresses: the hand-scheduled loop takes them as they are)
    const unsigned lds0 = (unsigned)(size_t)WK_LDS(smem);
    unsigned k_rd[8];
#pragma unroll
    for (int st = 0; st < 8; ++st) k_rd[st] = lds0 + kg * kTileBytes + col * 256 + (((2 * st + g) ^ (col & 15)) << 4);
    // V tile: row-major, chunk c of key k at slot c ^ ((k & 3) << 2).  The transpose read hands lane
    // i of a 16-lane group element (i & 3) of source lane 4*j + (i >> 2), j = 0..3.  Source lane p of
    // group u points at key 16*ks + 8*tt + 4*g + (p >> 2), features 32*blk + 16*(u&1) + 4*(p&3) .. +3,
    // so lane i receives feature 32*blk + 16*(u&1) + i of keys 16*ks + 8*tt + 4*g + 0..3: the four
    // k slots that registers 4*tt .. 4*tt+3 of the P^T operand of step ks stand for.
    //   address = v_rd[blk] + stage*16384 + ks*4096 + tt*2048
    unsigned v_rd[4];
    {
        const int u = lane >> 4, p = lane & 15;
#pragma unroll
        for (int blk = 0; blk < 4; ++blk)
            v_rd[blk] = lds0 + kVRing + kg * kTileBytes + (4 * g + (p >> 2)) * 256 +
                        ((4 * (blk ^ (p >> 2)) + 2 * (u & 1) + ((p & 3) >> 1)) << 4) + 8 * (p & 1);
    }
    // tile loads: wave w fills 1 KB blocks NB*w .. NB*w + NB-1 of the K tile and of the V tile; lane l
    // of a block lands in 16-byte slot l = (row r = l >> 4 of the block, slot p = l & 15)
    unsigned k_src[NB], v_src[NB];
    {
        const int r = lane >> 4, p = lane & 15;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int R = 4 * (NB * wave + i) + r;
            k_src[i] = R * 256 + ((p ^ (R & 15)) << 4);
            v_src[i] = R * 256 + ((p ^ (r << 2)) << 4);
        }
    }
    const char *Kh = win.K + (size_t)h * win.stride * 256;
    const char *Vh = a.V + (size_t)h * win.stride * 256;
    const unsigned last_off = (unsigned)(n_kv - 1) * 256u;
    char *const dma_dst = smem + wave * (NB * 1024);   // + slot*16384 (+ kVRing) + i*1024

    // Loads: NB per wave for a K tile, NB for a V tile (rel = tile index relative to t0).  Rows past the
    // window clamp to the last key; those keys are masked (weight exactly 0) before they can contribute.
    // IN_PLACE: one cursor walks the segment list in steps of a tile, at the K loads, which lead
    // everything else.  What later stages need of a tile is kept from the moment its K tile was requested:
    // the V tile is requested one K request later (two-deep line of its address and bounds) and S^T of
    // the tile is formed three K requests later (four-deep line of its number of valid keys).  Moving past
    // the list's last tile leaves the cursor on it (the look-ahead fetches it again and nobody reads it).
    // All of this is wave-uniform scalar state.
    struct TileRef { const char *base; int row, len; };
    const char *cur_k = nullptr, *cur_v = nullptr;
    int cur_len = 0, cur_row = 0, cur_seg = 0;
    TileRef v_line[2] = {{nullptr, 0, 0}, {nullptr, 0, 0}};
    unsigned valid_line = 0;   // four entries of 8 bits, newest lowest: valid keys of a tile, capped at 64 (scalar registers are scarce here)
    if constexpr (IN_PLACE) {
        if (n_seg > 0) {
            cur_len = __builtin_amdgcn_readfirstlane(seg_list[0].len);
            cur_k = uniform_ptr(seg_list[0].K);
            cur_v = uniform_ptr(seg_list[0].V);
        }
    }
    // one tile: rows past the segment's end clamp to its last row (those keys are masked when consumed)
    auto issue_at = [&](const char *base, int row, int len, const unsigned (&src)[NB], char *dst) {
        const unsigned t_off = (unsigned)row * 256u;
        if (row + kKeys <= len) {
#pragma unroll
            for (int i = 0; i < NB; ++i)
                __builtin_amdgcn_global_load_lds(WK_GLB(base + (t_off + src[i])), WK_LDS(dst + i * 1024), 16, 0, 0);
        } else {
            const unsigned seg_last = (unsigned)(len - 1) * 256u;
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const unsigned o = min(t_off + src[i], seg_last + (src[i] & 255u));
                __builtin_amdgcn_global_load_lds(WK_GLB(base + o), WK_LDS(dst + i * 1024), 16, 0, 0);
            }
        }
    };
    auto issue_k_in_place = [&](char *dst) {
        issue_at(cur_k, cur_row, cur_len, k_src, dst);
        v_line[1] = v_line[0];
        v_line[0] = TileRef{cur_v, cur_row, cur_len};
        valid_line = (valid_line << 8) | (unsigned)min(cur_len - cur_row, kKeys);   // 64: a full tile
        if (cur_row + kKeys < cur_len) {
            cur_row += kKeys;
        } else if (cur_seg + 1 < n_seg) {
            ++cur_seg;
            cur_row = 0;
            cur_len = __builtin_amdgcn_readfirstlane(seg_list[cur_seg].len);
            cur_k = uniform_ptr(seg_list[cur_seg].K);
            cur_v = uniform_ptr(seg_list[cur_seg].V);
        }
    };
    auto issue_k = [&](int rel, int slot) {
        const unsigned t_off = (unsigned)(t0 + rel) * (kKeys * 256u);
        char *dst = dma_dst + slot * kTileBytes;
        if constexpr (IN_PLACE) {
            issue_k_in_place(dst);
            return;
        }
        if ((t0 + rel + 1) * kKeys <= n_kv) {
#pragma unroll
            for (int i = 0; i < NB; ++i)
                __builtin_amdgcn_global_load_lds(WK_GLB(Kh + skip_gap(t_off + k_src[i])), WK_LDS(dst + i * 1024), 16, 0, 0);
        } else {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const unsigned ko = min(t_off + k_src[i], last_off + (k_src[i] & 255u));
                __builtin_amdgcn_global_load_lds(WK_GLB(Kh + skip_gap(ko)), WK_LDS(dst + i * 1024), 16, 0, 0);
            }
        }
    };
    auto issue_v = [&](int rel, int slot, const TileRef &ref) {   // ref: where the tile is (IN_PLACE)
        const unsigned t_off = (unsigned)(t0 + rel) * (kKeys * 256u);
        char *dst = dma_dst + slot * kTileBytes + kVRing;
        if constexpr (IN_PLACE) {
            issue_at(ref.base, ref.row, ref.len, v_src, dst);
            return;
        }
        if ((t0 + rel + 1) * kKeys <= n_kv) {
#pragma unroll
            for (int i = 0; i < NB; ++i)
                __builtin_amdgcn_global_load_lds(WK_GLB(Vh + skip_gap(t_off + v_src[i])), WK_LDS(dst + i * 1024), 16, 0, 0);
        } else {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const unsigned vo = min(t_off + v_src[i], last_off + (v_src[i] & 255u));
                __builtin_amdgcn_global_load_lds(WK_GLB(Vh + skip_gap(vo)), WK_LDS(dst + i * 1024), 16, 0, 0);
            }
        }
    };

    f32x16 o[4];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[b][r] = 0.f;
    float m_run = -FLT_MAX;         // what probabilities are relative to, in scaled (log2) units; finite for the sake of scores of -inf, as in k_attn_f32
    float l_run[2] = {0.f, 0.f};    // row sums over the even and the odd tiles (KG == 2: this wave group's, and nothing)
    const float c_log2 = a.scale_log2;

    auto compute_s = [&](int byte_off, f32x16 (&s)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[b][r] = 0.f;
        // the 32-key blocks are independent accumulation chains: alternate them
#pragma unroll
        for (int st = 0; st < 8; ++st)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const bf16x8 ka = *WK_LDS_AT(const bf16x8, k_rd[st] + byte_off + b * 8192);
                s[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qb[st], s[b], 0, 0, 0);
            }
    };
    // IN_PLACE: the tile whose S^T has just been formed had its K tile requested three requests ago; keys
    // past its segment's end get -inf (weight exactly 0).
    auto mask_segment_tail = [&](f32x16 (&s)[2]) __attribute__((always_inline)) {
        const int valid = (int)((valid_line >> (24 - 8 * kg)) & 255u);
        if (valid < kKeys) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (32 * b + 8 * (r >> 2) + 4 * g + (r & 3) >= valid) s[b][r] = -INFINITY;
        }
    };
    // scaled row max of a tile's raw logits (both lane halves combined)
    auto tile_max = [&](const f32x16 (&s)[2]) __attribute__((always_inline)) {
        float mx[10];
#pragma unroll
        for (int i = 0; i < 10; ++i) {
            const int e = 3 * i;
            mx[i] = max3(s[e >> 4][e & 15], s[(e + 1) >> 4][(e + 1) & 15], s[(e + 2) >> 4][(e + 2) & 15]);
        }
        float m = max3(max3(mx[0], mx[1], mx[2]), max3(mx[3], mx[4], mx[5]), max3(mx[6], mx[7], mx[8]));
        m = max3(m, mx[9], fmaxf(s[1][14], s[1][15]));
        return max_across_halves(m) * c_log2;
    };
    // lazy rescale: the running max only moves when some row's max grew by more than 2^8
    auto maybe_rescale = [&](float m_tile) __attribute__((always_inline)) {
        if (__any(m_tile > m_run + 8.0f)) {
            const float m_new = fmaxf(m_run, m_tile);
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
            m_run = m_new;
            l_run[0] *= alpha;
            if constexpr (KG == 1) l_run[1] *= alpha;
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[b][r] *= alpha;
        }
    };
    // p = exp2(s*c - m) rounded to bf16; registers 8*t2 .. 8*t2+7 of block b -> k step 2*b + t2.
    // The row sum uses the rounded probabilities, the ones the P V product sees.  Even and odd tiles are summed apart,
    // as the two wave groups of KG == 2 do: the log-sum-exp is then the same in every layout of the launch, as long as the key range
    // is not split, no row's maximum grows by more than 2^8 behind the first tile and no lane's sum reaches 2^24 (what the groups weigh keys against then parts).
    auto probabilities = [&](const f32x16 (&s)[2], bf16x8 (&pb)[4], float &l_sum) __attribute__((always_inline)) {
        const float neg_m = -m_run;
        const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    const float p0 = __builtin_amdgcn_exp2f(fmaf(s[b][8 * t2 + e], c_log2, neg_m));
                    const float p1 = __builtin_amdgcn_exp2f(fmaf(s[b][8 * t2 + e + 1], c_log2, neg_m));
                    const bf16x2 pk = __builtin_convertvector(f32x2{p0, p1}, bf16x2);
                    pb[2 * b + t2][e] = pk[0];
                    pb[2 * b + t2][e + 1] = pk[1];
                    l_sum = __builtin_amdgcn_fdot2_f32_bf16(pk, ones, l_sum, false);
                }
    };
    auto accumulate_pv = [&](int byte_off, const bf16x8 (&pb)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const unsigned p = v_rd[b] + byte_off + ks * 4096;
                const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(WK_LDS_AT(i16x4, p));
                const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(WK_LDS_AT(i16x4, p + 2048));
                const i16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                o[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), pb[ks], o[b], 0, 0, 0);
            }
    };

    // The ring slot of tile j is j & 3.  Whole trips round the ring come first (the steady state), then the left-over
    // steps, then the last tile (pair) at whatever ring position that leaves it.
    // KG == 1: step j multiplies K tile j+1 (S^T one step early) and V tile j, so K runs one tile ahead of V:
    // it loads K tile j+4 into the slot of K tile j (read in step j-1) and V tile j+3 into the slot of V tile j-1.
    // Both then have three steps to land before the step that needs them.
    // KG == 2: step j multiplies K tiles 2j+2, 2j+3 and V tiles 2j, 2j+1 (wave group kg one of each) and loads K tiles
    // 2j+4, 2j+5 and V tiles 2j+2, 2j+3 into the slots read in step j-1: one step to land.
    const int n_steps = KG == 1 ? t1 - t0 - 1 : (t1 - t0 + 1) / 2 - 1;
    auto issue_step = [&](int j, const int POS) __attribute__((always_inline)) {   // POS: ring slot of the step's first V tile
        if constexpr (KG == 1) {
            issue_k(j + 4, POS);
            issue_v(j + 3, (POS + 3) & 3, v_line[1]);
        } else {
            issue_v(2 * j + 2, (POS + 2) & 3, v_line[1]);
            issue_v(2 * j + 3, (POS + 3) & 3, v_line[0]);
            issue_k(2 * j + 4, POS);
            issue_k(2 * j + 5, POS + 1);
        }
    };
    auto ring_pos = [](int j) { return KG == 1 ? j & 3 : (2 * j) & 3; };
    auto end_step = [&]() __attribute__((always_inline)) {
        // KG == 1: all but the loads of this step and the one before have landed
        __builtin_amdgcn_s_waitcnt(KG == 1 ? kWaitTwoSteps : kWaitAll);
        __syncthreads();
    };
    constexpr bool kTrips = TRIPS && QW * KG == 8;
    // Trips of the hand-scheduled loop: the steps behind them stay in C++, which are the last whole trips, whose loads are clamped to the window, the
    // left-over steps and the last, possibly partial tile.  (IN_PLACE: the most there can be; where they run is seen on the way.)
    const int n_trips = IN_PLACE ? n_steps / (4 / KG) : min((n_kv / kKeys - 4 - t0) / 4, n_steps / (4 / KG));
    // (One trip is still as good as none: 40 heads x 1,000 queries x 512 keys 19.9 us with it, 20.3 without, x 700 24.0 and 24.2, 40 x 4,680 x 512 69.7 and 70.0, x 600 78.5
    // and 78.0, x 700 83.3 and 82.9; in pairs of tiles, where it is two steps, 5 x 392 x 615 15.0 and 15.0.)
    const bool may_lose = kTrips && n_trips > 0;   // of the whole workgroup
    int *const lost = reinterpret_cast<int *>(smem + kRings + 512);
    if (may_lose && tid == 0) *lost = 0;   // (barriers lie between)
    issue_k(0, 0);
    issue_k(1, 1);
    issue_v(0, 0, v_line[1]);
    if constexpr (KG == 1) {
        issue_k(2, 2);
        issue_v(1, 1, v_line[1]);
        issue_k(3, 3);
        issue_v(2, 2, v_line[1]);
    } else {
        issue_v(1, 1, v_line[0]);
        issue_k(2, 2);
        issue_k(3, 3);
    }
    // KG == 1: K tiles 0, 1 and V tile 0 of this wave have landed; KG == 2: K tiles 0 and 1 (and V tile 0 or the like)
    __builtin_amdgcn_s_waitcnt(kWaitTwoSteps);
    __syncthreads();
    if (qt * (QW * 32) + qw * 32 >= a.N_q) {
        // A wave whose 32 queries all lie past N_q (last query tile of a head): it keeps loading its
        // share of every tile and meets every barrier, but leaves the matrix and vector pipes of its
        // SIMD to the wave that has work.
        if constexpr (KG == 2) __builtin_amdgcn_s_waitcnt(kWaitAll);
        __syncthreads();   // the others' first S^T has been formed from K tile 0
        for (int j = 0; j < n_steps; ++j) {
            issue_step(j, ring_pos(j));
            end_step();
        }
        __builtin_amdgcn_s_waitcnt(kWaitAll);
        if (KG == 2 || may_lose) __syncthreads();   // as at the end of a pass
        if (may_lose && __builtin_amdgcn_readfirstlane(*lost) != 0) return true;
        if constexpr (KG == 2) __syncthreads();   // the wave groups' meeting
        return false;
    }
    f32x16 s_a[2], s_b[2];   // S^T of tiles at even / odd ring positions
    float mt;
    compute_s(0, s_a);
    if constexpr (IN_PLACE) mask_segment_tail(s_a);
    mt = tile_max(s_a);
    float *const m_first = reinterpret_cast<float *>(smem + kRings) + qw * 32 + col;
    if constexpr (KG == 2) {
        if (kg == 0) *m_first = mt;
        __builtin_amdgcn_s_waitcnt(kWaitAll);   // everything requested so far is read in step 0
    }
    __syncthreads();   // the first K tile (pair) has been read by every wave: step 0 may load into its slot

    // from the first tile's maximum on, both wave groups as a wave that walks every tile
    m_run = fmaxf(KG == 2 ? *m_first : mt, -FLT_MAX);

    // one pipeline step: this wave's tile at ring position POS (+ kg) is consumed, S^T of its next tile produced
    auto step = [&](int j, const int POS, f32x16 (&s_cur)[2], f32x16 (&s_next)[2], float &l_sum)
        __attribute__((always_inline)) {
        issue_step(j, POS);
        maybe_rescale(mt);
        compute_s(((POS + KG) & 3) * kTileBytes, s_next);
        bf16x8 pb[4];
        probabilities(s_cur, pb, l_sum);
        // (the rare branch sits between the two matrix products, so that the row max below can still be
        // interleaved with the second one)
        if constexpr (IN_PLACE) mask_segment_tail(s_next);
        accumulate_pv(POS * kTileBytes, pb);
        mt = tile_max(s_next);
        end_step();
    };
    int j = 0;
    bool tripped = false;
    // Whole trips round the ring in a hand-scheduled loop (written by gen_attn_loop.py, which documents its schedule and register map), whose
    // look-ahead loads must all lie in full tiles of one array: K tiles from k_base + koff on, V tiles from v_base + voff on.  It is
    // the four (KG == 2: two) `step`s below in what it computes -- same ring protocol, same arithmetic in the same order -- except
    // that the maximum does not run: the reference goes up by a power of two, 2^63 at most, when a row sum has reached 2^24.  Its operands
    // are pinned to the registers its text names.  Without the maximum, and with its vector work dealt over 22 of a step's 32 products, 40 heads x
    // 4,680 queries x 28,080 keys 2,256 -> 2,155 us, 12 x 2,640 x 10,560 156.8 -> 151.9, 12 x 2,640 x 211,200 3,044 -> 2,933.
    auto trips = [&](int G, const char *k_base, const char *v_base, unsigned koff, unsigned voff) __attribute__((always_inline)) {
        if constexpr (QW * KG == 8) {
            // the tile with the first row behind the gap, and the steps up to the one that requests its K tile
            const unsigned gap_tile = gap_from / kTileBytes * kTileBytes;
            int gap_steps = (((int)(gap_from / kTileBytes) - t0 - 4) >> (KG - 1)) + 2;
            if constexpr (GAP) {
                if (koff > gap_tile) koff += gap_bytes;
                if (voff > gap_tile) voff += gap_bytes;
            }
            else {
                k_base += koff;
                v_base += voff;
            }
            const unsigned dst = (unsigned)(size_t)WK_LDS(dma_dst);
            int g_left = G;
            const bf16x8 q0 = qb[0], q1 = qb[1], q2 = qb[2], q3 = qb[3], q4 = qb[4], q5 = qb[5], q6 = qb[6], q7 = qb[7];
            f32x16 o0 = o[0], o1 = o[1], o2 = o[2], o3 = o[3], sa0 = s_a[0], sa1 = s_a[1];
            const unsigned ks0 = k_src[0], ks1 = k_src[NB - 1], vs0 = v_src[0], vs1 = v_src[NB - 1];
#define WK_ATTN_LOOP_OUT "+{v[0:15]}"(o0), "+{v[16:31]}"(o1), "+{v[32:47]}"(o2), "+{v[48:63]}"(o3), "+{v[64:79]}"(sa0), \
                  "+{v[80:95]}"(sa1), "+{v240}"(m_run), "+{v241}"(l_run[0]), "+{v242}"(l_run[1]), "+{s44}"(g_left), \
                  "+{s[36:37]}"(k_base), "+{s[38:39]}"(v_base)
#define WK_ATTN_LOOP_IN "{v[128:131]}"(q0), "{v[132:135]}"(q1), "{v[136:139]}"(q2), "{v[140:143]}"(q3), "{v[144:147]}"(q4), \
                  "{v[148:151]}"(q5), "{v[152:155]}"(q6), "{v[156:159]}"(q7), "{v224}"(k_rd[0]), "{v225}"(k_rd[1]), \
                  "{v226}"(k_rd[2]), "{v227}"(k_rd[3]), "{v228}"(k_rd[4]), "{v229}"(k_rd[5]), "{v230}"(k_rd[6]), "{v231}"(k_rd[7]), \
                  "{v232}"(v_rd[0]), "{v233}"(v_rd[1]), "{v234}"(v_rd[2]), "{v235}"(v_rd[3]), "{v236}"(ks0), "{v237}"(ks1), \
                  "{v238}"(vs0), "{v239}"(vs1), "{s42}"(dst), "{s43}"(c_log2)
            if constexpr (GAP && KG == 1) {
                asm volatile(
#include "wk_attn_gap_loop_gfx950.inc"
                    : WK_ATTN_LOOP_OUT, "+{s40}"(koff), "+{s41}"(voff), "+{s49}"(gap_steps)
                    : WK_ATTN_LOOP_IN, "{s46}"(gap_from), "{s47}"(gap_bytes), "{s48}"(gap_tile)
                    : WK_ATTN_LOOP_CLOBBERS, "s45", "vcc", "memory");
            } else if constexpr (GAP) {
                asm volatile(
#include "wk_attn_gap_pair_loop_gfx950.inc"
                    : WK_ATTN_LOOP_OUT, "+{s40}"(koff), "+{s41}"(voff), "+{s49}"(gap_steps)
                    : WK_ATTN_LOOP_IN, "{s46}"(gap_from), "{s47}"(gap_bytes), "{s48}"(gap_tile)
                    : WK_ATTN_LOOP_CLOBBERS, "s45", "vcc", "memory");
            } else if constexpr (KG == 1) {
                asm volatile(
#include "wk_attn_loop_gfx950.inc"
                    : WK_ATTN_LOOP_OUT : WK_ATTN_LOOP_IN : WK_ATTN_LOOP_CLOBBERS, "s45", "vcc", "memory");
            } else {
                asm volatile(
#include "wk_attn_pair_loop_gfx950.inc"
                    : WK_ATTN_LOOP_OUT : WK_ATTN_LOOP_IN : WK_ATTN_LOOP_CLOBBERS, "s45", "vcc", "memory");
            }
            o[0] = o0; o[1] = o1; o[2] = o2; o[3] = o3; s_a[0] = sa0; s_a[1] = sa1;
            mt = tile_max(s_a);
            tripped = true;
            // row sums that have grown are brought below 1 here too (from 2^63 at most, as in the loop: exp2 gives 0 below -126), so that the reference is near the
            // maximum where it is compared with others
            if (__any(l_run[0] + l_run[1] >= 0x1p24f)) {
                const auto e = __builtin_amdgcn_permlane32_swap(__builtin_amdgcn_frexp_expf(l_run[0] + l_run[1]),
                                                                __builtin_amdgcn_frexp_expf(l_run[0] + l_run[1]), false, false);
                const float m_new = m_run + (float)min(max(max((int)e[0], (int)e[1]), 0), 63), alpha = __builtin_amdgcn_exp2f(m_run - m_new);
                m_run = m_new;
                l_run[0] *= alpha;
                l_run[1] *= alpha;
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[b][r] *= alpha;
            }
            j += G * (4 / KG);
        }
    };
    if constexpr (kTrips && !IN_PLACE) {
        if (n_trips > 0) trips(n_trips, Kh, Vh, (unsigned)(t0 + 4) * kTileBytes, (unsigned)(t0 + 4 - KG) * kTileBytes);
    }
    // IN_PLACE: the trips whose tiles -- from the ones whose S^T comes next to the last one requested -- are full and of the cursor's segment, and
    // leave the cursor in it.  The steps across a segment's boundary stay in C++.
    auto trips_in_segment = [&]() __attribute__((always_inline)) {
        if constexpr (IN_PLACE && kTrips) {
            constexpr unsigned kAhead = KG == 1 ? 0x404040u : 0x4040u;   // tiles j+1 to j+3, KG == 2: 2j+2 and 2j+3
            if ((valid_line & (KG == 1 ? 0xffffffu : 0xffffu)) != kAhead) return;
            if (cur_row < KG * kKeys || v_line[0].base != cur_v || v_line[0].row + kKeys != cur_row) return;
            if (KG == 2 && (v_line[1].base != cur_v || v_line[1].row + 2 * kKeys != cur_row)) return;
            const int G = min((cur_len - cur_row - 1) / kKeys / 4, (n_steps - j) / (4 / KG));
            if (G <= 0) return;
            trips(G, cur_k, cur_v, (unsigned)cur_row * 256u, (unsigned)(cur_row - KG * kKeys) * 256u);
            cur_row += 4 * G * kKeys;
            v_line[0] = TileRef{cur_v, cur_row - kKeys, cur_len};
            v_line[1] = TileRef{cur_v, cur_row - 2 * kKeys, cur_len};
            valid_line = 0x40404040u;
        }
    };
    if constexpr (KG == 1) {
        for (; j + 4 <= n_steps; j += 4) {
            trips_in_segment();
            if (IN_PLACE && TRIPS && j + 4 > n_steps) break;
            step(j, 0, s_a, s_b, l_run[0]);
            step(j + 1, 1, s_b, s_a, l_run[1]);
            step(j + 2, 2, s_a, s_b, l_run[0]);
            step(j + 3, 3, s_b, s_a, l_run[1]);
        }
    } else {
        for (; j + 2 <= n_steps; j += 2) {
            trips_in_segment();
            if (IN_PLACE && TRIPS && j + 2 > n_steps) break;
            step(j, 0, s_a, s_b, l_run[0]);
            step(j + 1, 2, s_b, s_a, l_run[0]);
        }
    }
    // last tile (ring position POS): the only one that can be partial.  Mask the keys past the window and
    // redo its max.
    auto last_tile = [&](const int POS, f32x16 (&s_cur)[2], float &l_sum) __attribute__((always_inline)) {
        const int kt = KG == 1 ? (t1 - 1) * kKeys : (t0 + 2 * n_steps + kg) * kKeys;
        if (!IN_PLACE && kt + kKeys > n_kv) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int key = kt + 32 * b + 8 * (r >> 2) + 4 * g + (r & 3);
                    if (key >= n_kv) s_cur[b][r] = -INFINITY;
                }
            mt = tile_max(s_cur);
        }
        maybe_rescale(mt);
        bf16x8 pb[4];
        probabilities(s_cur, pb, l_sum);
        accumulate_pv(POS * kTileBytes, pb);
    };
    // the left-over steps and the last tile: one copy of the code, ring position at run time,
    // S^T handed back to s_a (and the sum of the next tile's parity to l_run[0]) after each step
    for (; j < n_steps; ++j) {
        step(j, ring_pos(j), s_a, s_b, l_run[0]);
#pragma unroll
        for (int b = 0; b < 2; ++b) s_a[b] = s_b[b];
        if constexpr (KG == 1) {
            const float t = l_run[0];
            l_run[0] = l_run[1];
            l_run[1] = t;
        }
    }
    // (an odd count of tiles leaves the second wave group without one: what lies behind the range -- the next range's rows, or
    // the last row again -- has no part in this one)
    if (KG == 1 || kg == 0 || (t1 - t0) % 2 == 0) last_tile(ring_pos(n_steps), s_a, l_run[0]);
    __builtin_amdgcn_s_waitcnt(0x0F70);   // drain the clamped look-ahead loads before the LDS is released
    bool wave_lost = false;
    if constexpr (kTrips)
        if (tripped) {
            // The bits of the largest magnitude, or of NaN where there is one.  In assembly, and looked at as bits, because the compiler takes no number here
            // for NaN; and behind a wait for O^T's matrix instructions, which it does not put in front of assembly.
            unsigned top = __float_as_uint(l_run[0] + l_run[1]);
            asm("s_nop 7\n\ts_nop 7" : "+v"(o[0]), "+v"(o[1]), "+v"(o[2]), "+v"(o[3]));
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const f32x16 &x = o[b];
                asm("v_maximum3_f32 %0, %0, |%1|, |%2|\n\tv_maximum3_f32 %0, %0, |%3|, |%4|\n\tv_maximum3_f32 %0, %0, |%5|, |%6|\n\t"
                    "v_maximum3_f32 %0, %0, |%7|, |%8|\n\tv_maximum3_f32 %0, %0, |%9|, |%10|\n\tv_maximum3_f32 %0, %0, |%11|, |%12|\n\t"
                    "v_maximum3_f32 %0, %0, |%13|, |%14|\n\tv_maximum3_f32 %0, %0, |%15|, |%16|"
                    : "+v"(top)
                    : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(x[6]), "v"(x[7]), "v"(x[8]), "v"(x[9]), "v"(x[10]),
                      "v"(x[11]), "v"(x[12]), "v"(x[13]), "v"(x[14]), "v"(x[15]));
            }
            wave_lost = __any((top & 0x7fffffffu) >= 0x7f800000u);
            if (wave_lost) *lost = 1;
        }
    if constexpr (KG == 2) {
        __syncthreads();   // every wave has read its last tile and its look-ahead loads have landed
        if (may_lose && __builtin_amdgcn_readfirstlane(*lost) != 0) return true;
        // The wave groups meet: waves 4..7 leave (O^T, max, sum) of their keys in the ring, waves 0..3 add it to theirs.
        // Register r of a wave's lane sits at [qw][r][lane]: consecutive lanes, consecutive banks.
        float *meet = reinterpret_cast<float *>(smem) + qw * (66 * 64) + lane;
        if (kg == 1) {
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) meet[(16 * b + r) * 64] = o[b][r];
            meet[64 * 64] = m_run;
            meet[65 * 64] = l_run[0];
        }
        __syncthreads();
        if (kg == 1) return false;
        const float m_other = meet[64 * 64];
        const float m_new = fmaxf(m_run, m_other);
        const float w0 = __builtin_amdgcn_exp2f(m_run - m_new), w1 = __builtin_amdgcn_exp2f(m_other - m_new);
        m_run = m_new;
        l_run[0] *= w0;
        l_run[1] = w1 * meet[65 * 64];
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[b][r] = fmaf(w1, meet[(16 * b + r) * 64], w0 * o[b][r]);
    }
    const float l_lane = l_run[0] + l_run[1];
    const float l_tot = l_lane + __shfl_xor(l_lane, 32);
    const bool store = q_ok && !wave_lost && !stored;
    if (store && !partial_out) {
        const size_t qrow = out_row();
        char *Orow = a.O + qrow * 256;
        const float inv = 1.f / l_tot;
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int dv = 32 * b + 8 * t + 4 * g;
                const bf16x2 lo = __builtin_convertvector(f32x2{o[b][4 * t] * inv, o[b][4 * t + 1] * inv}, bf16x2);
                const bf16x2 hi = __builtin_convertvector(f32x2{o[b][4 * t + 2] * inv, o[b][4 * t + 3] * inv}, bf16x2);
                uint2 w;
                w.x = __builtin_bit_cast(uint32_t, lo);
                w.y = __builtin_bit_cast(uint32_t, hi);
                *reinterpret_cast<uint2 *>(Orow + dv * 2) = w;
            }
        if (lse && g == 0) lse[qrow] = (m_run + log2f(l_tot)) * 0.6931471805599453f;
    } else if (store) {   // partial result of this key range, merged by k_attn_merge
        const size_t prow = part_row();
        float *Po = a.part_o + prow * WK_D;
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                *reinterpret_cast<float4 *>(Po + 32 * b + 8 * t + 4 * g) =
                    float4{o[b][4 * t], o[b][4 * t + 1], o[b][4 * t + 2], o[b][4 * t + 3]};
        if (g == 0) { a.part_ml[prow * 2] = m_run; a.part_ml[prow * 2 + 1] = l_tot; }
    }
    // Waves that walk every tile meet behind their stores: the older wave of each SIMD is done hundreds of cycles before the younger one, and in front of its
    // stores that was lost to every workgroup (40 heads x 4,680 queries x 900 keys 102.6 -> 101.0 us, x 1,000 108.3 -> 106.7, of a kernel with a running maximum and no such
    // meeting 101.9 and 107.2)
    if (KG == 1 && may_lose) {
        stored = !wave_lost;
        __syncthreads();   // every wave has read its last tile and its look-ahead loads have landed
        return __builtin_amdgcn_readfirstlane(*lost) != 0;
    }
    return false;
}

// A second pass, in the compiled steps with their running maximum, begins anew from the arguments: whatever the first one had in registers
// need not outlive it (kept for the second, 70 registers were in scratch around the loop).
// Scores that grow by more than 2^100 or so behind the first tile, and windows that hold infinities, take both: 12 heads x 2,640 queries x 10,560 keys
// 163 us with a running maximum in the loop, 337; all others 152 instead of 157.
template <int QW, int KG, bool MULTI, bool IN_PLACE, bool GAP = false, bool TRIPS = !IN_PLACE>
__global__ __launch_bounds__(QW * KG * 64, 2) void k_attn_bf16(AttnArgs a, SubTable sub) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    bool stored = false;
    if (!attend<QW, KG, MULTI, IN_PLACE, GAP, TRIPS>(a, sub, wave, stored)) return;
    if constexpr (TRIPS && QW * KG == 8) {
        struct Args { AttnArgs a; SubTable sub; };
        auto args = (const __attribute__((address_space(4))) Args *)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(args));
        const Args *const again = (const Args *)args;
        attend<QW, KG, MULTI, IN_PLACE, GAP, false>(again->a, again->sub, wave, stored);
    }
}

// ------------------------------------------------------------------------------------------
// Log-sum-exp only (a.O == NULL; query-based retrieval, paper Sec. 4.2 / App. C).  Without the
// P V product the matrix work halves while the exp2 work per key stays, so the kernel is bound
// by the VALU, not by the matrix cores.  It therefore drops the in-wave software pipeline of
// k_attn_bf16 (two S^T tiles in registers) for occupancy: under 128 VGPRs and with a 64 KB K
// ring, two workgroups = four waves per SIMD share a CU, and one wave's MFMAs run under the
// others' exp2; the workgroup's waves meet at a barrier only every second tile.  Same tile layout,
// loads and arithmetic (bf16-rounded probabilities summed by
// dot2) as the full kernel: the lse values are bit-identical to those wk_attention returns
// beside O, as long as that call does not split the key range, no row's maximum grows by more than 2^8 behind the first tile and no lane's row sum reaches
// 2^24 there (which takes 2^16 keys of a lane's that weigh 2^8 each, or growth).
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(512, 4) void k_lse_bf16(AttnArgs a) {
    extern __shared__ __attribute__((aligned(256))) char smem[];
    int c, h, qt, sp;
    if (!work_item(a, c, h, qt, sp)) return;
    const Window win = window_of(a, c);
    const int n_kv = win.n_kv;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, g = lane >> 5;
    const int q = qt * 256 + wave * 32 + col;
    const bool q_ok = q < a.N_q;
    const int q_ld = q_ok ? q : a.N_q - 1;
    const char *Qrow = a.Q + ((size_t)h * a.q_rows + a.q_off + q_ld) * 256;
    float *const out = win.lse + (size_t)h * a.q_rows + a.q_off + q;
    if (n_kv == 0) {
        if (q_ok && g == 0) *out = -INFINITY;
        return;
    }
    bf16x8 qb[8];
#pragma unroll
    for (int st = 0; st < 8; ++st) qb[st] = *reinterpret_cast<const bf16x8 *>(Qrow + (2 * st + g) * 16);
    unsigned k_rd[8];   // as in k_attn_bf16: chunk 2*st + g of key col, slot c ^ (key & 15)
#pragma unroll
    for (int st = 0; st < 8; ++st) k_rd[st] = (unsigned)(size_t)WK_LDS(smem) + col * 256 + (((2 * st + g) ^ (col & 15)) << 4);
    unsigned k_src[2];
    {
        const int r = lane >> 4, p = lane & 15;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int R = 4 * (2 * wave + i) + r;
            k_src[i] = R * 256 + ((p ^ (R & 15)) << 4);
        }
    }
    const char *Kh = win.K + (size_t)h * win.stride * 256;
    const unsigned last_off = (unsigned)(n_kv - 1) * 256u;
    char *const dma_dst = smem + wave * 2048;
    // 2 loads per wave and tile; tiles that end past the window (also the look-ahead past the last
    // tile) clamp their rows to the last key
    auto issue_tile = [&](int t, int slot) {
        const unsigned t_off = (unsigned)t * (kKeys * 256u);
        char *dst = dma_dst + slot * kTileBytes;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const unsigned ko = min(t_off + k_src[i], last_off + (k_src[i] & 255u));
            __builtin_amdgcn_global_load_lds(WK_GLB(Kh + ko), WK_LDS(dst + i * 1024), 16, 0, 0);
        }
    };
    float m_run = -INFINITY;
    f32x2 l_run = {0.f, 0.f};   // row sums of the even and the odd tiles, apart as in k_attn_bf16
    const float c_log2 = a.scale_log2;
    auto tile = [&](int byte_off, int kt, bool partial, auto odd_tag) __attribute__((always_inline)) {
        f32x16 s[2];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[b][r] = 0.f;
#pragma unroll
        for (int st = 0; st < 8; ++st)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const bf16x8 ka = *WK_LDS_AT(const bf16x8, k_rd[st] + byte_off + b * 8192);
                s[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qb[st], s[b], 0, 0, 0);
            }
        if (partial) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int key = kt + 32 * b + 8 * (r >> 2) + 4 * g + (r & 3);
                    if (key >= n_kv) s[b][r] = -INFINITY;
                }
        }
        float mx[10];
#pragma unroll
        for (int i = 0; i < 10; ++i) {
            const int e = 3 * i;
            mx[i] = max3(s[e >> 4][e & 15], s[(e + 1) >> 4][(e + 1) & 15], s[(e + 2) >> 4][(e + 2) & 15]);
        }
        float m = max3(max3(mx[0], mx[1], mx[2]), max3(mx[3], mx[4], mx[5]), max3(mx[6], mx[7], mx[8]));
        m = max3(m, mx[9], fmaxf(s[1][14], s[1][15]));
        const float mt = max_across_halves(m) * c_log2;
        if (__any(mt > m_run + 8.0f)) {   // lazy rescale, as in k_attn_bf16
            const float m_new = fmaxf(m_run, mt);
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
            l_run[0] *= alpha;
            l_run[1] *= alpha;
            m_run = m_new;
        }
        float l_tile = l_run[decltype(odd_tag)::value];
        const float neg_m = -m_run;
        const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 16; e += 2) {
                const float p0 = __builtin_amdgcn_exp2f(fmaf(s[b][e], c_log2, neg_m));
                const float p1 = __builtin_amdgcn_exp2f(fmaf(s[b][e + 1], c_log2, neg_m));
                l_tile = __builtin_amdgcn_fdot2_f32_bf16(__builtin_convertvector(f32x2{p0, p1}, bf16x2), ones, l_tile,
                                                         false);
            }
        l_run[decltype(odd_tag)::value] = l_tile;
    };
    const int n_full = n_kv / kKeys;   // full tiles; one partial tile may follow
    const bool tail = n_full * kKeys < n_kv;
    issue_tile(0, 0);
    issue_tile(1, 1);
    // One barrier per two tiles.  Before it, this wave's loads of tiles j and j+1 have landed
    // (vmcnt(0): nothing newer is in flight yet); behind it every wave is done with tiles j-2 and
    // j-1, whose slots tiles j+2 and j+3 may overwrite.
    auto open_pair = [&](int j, auto pos_tag) __attribute__((always_inline)) {
        constexpr int POS = decltype(pos_tag)::value;
        __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();
        issue_tile(j + 2, (POS + 2) & 3);
        issue_tile(j + 3, (POS + 3) & 3);
    };
    using P0 = std::integral_constant<int, 0>;
    using P2 = std::integral_constant<int, 2>;
    const bool idle = qt * 256 + wave * 32 >= a.N_q;   // no valid query in this wave: loads and barriers only
    auto full_pair = [&](int j, auto pos_tag) __attribute__((always_inline)) {
        constexpr int POS = decltype(pos_tag)::value;
        open_pair(j, pos_tag);
        if (idle) return;
        tile(POS * kTileBytes, j * kKeys, false, std::false_type{});
        tile((POS + 1) * kTileBytes, (j + 1) * kKeys, false, std::true_type{});
    };
    // what is left after the full pairs: at most one full tile and the partial one
    auto last_pair = [&](int j, auto pos_tag, int full) __attribute__((always_inline)) {
        constexpr int POS = decltype(pos_tag)::value;
        open_pair(j, pos_tag);
        if (idle) return;
        if (full) {
            tile(POS * kTileBytes, j * kKeys, false, std::false_type{});
            if (tail) tile((POS + 1) * kTileBytes, (j + 1) * kKeys, true, std::true_type{});
        } else {
            tile(POS * kTileBytes, j * kKeys, true, std::false_type{});
        }
    };
    int j = 0;
    for (; j + 4 <= n_full; j += 4) {
        full_pair(j, P0{});
        full_pair(j + 2, P2{});
    }
    int rest = n_full - j;   // 0..3 full tiles, then perhaps the partial one
    if (rest >= 2) {
        full_pair(j, P0{});
        j += 2;
        rest -= 2;
        if (rest || tail) last_pair(j, P2{}, rest);
    } else if (rest || tail) {
        last_pair(j, P0{}, rest);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);   // drain the clamped look-ahead loads before the LDS is released
    const float l_lane = l_run[0] + l_run[1];
    const float l_tot = l_lane + __shfl_xor(l_lane, 32);
    if (q_ok && g == 0) *out = (m_run + log2f(l_tot)) * 0.6931471805599453f;
}

// ------------------------------------------------------------------------------------------
// Log-sum-exp only, of longer windows (lse_wide): workgroups of four waves with 64 queries each, two workgroups (two waves
// per SIMD) on a compute unit, each with its own 64 KB ring of four K tiles.
//
// Bound by neither pipe alone: a tile of 64 queries has 1,024 cycles of matrix and 1,120 of vector instructions (an exp2 of a wave is 8, and a weight costs one, a
// multiply-add and halves of a rounding and of an add) and takes 1,790; beside full matrix pipes the mix would take 1,340.  So no row maxima are taken (24 of 112 vector instructions per 32 queries and tile): every score is weighed against
// the first tile's maximum of its row, and only where a lane's sum over a tile reaches 2^8 the tile's weights are added unrounded and
// the reference moves up (by a power of two, which changes no rounding).  A weight far above the others is thus exact, as it is
// with a maximum that moves; against 64 bits the error is 0.9 of k_lse_bf16's where keys stand out, and the same (to the bit) where
// no tile's sum grows that far.  Every K fragment read from LDS feeds two products.
// 120 chunks of 1,560 keys, 40 heads x 4,680 queries, both in turn on one box: 15.7 M cycles at 1.73 GHz, 8.99 ms (matrix pipe busy
// 57 %, vector pipe 62 %), k_lse_bf16 18.4 M at 1.79 GHz, 10.27 ms; this layout with the maxima 18.5 M.  Depths of the reads ahead and
// the place of the vector work change nothing (0.3 %) as long as it leaves no gap: without it beside a step's first three products 18.0 M.
// Nothing lies in scratch: three registers of query numbers that did wrote 265 MB a launch beside its 90 MB of results.
// ------------------------------------------------------------------------------------------
#define WK_LSE_LOOP_CLOBBERS \
    "v64", "v65", "v66", "v67", "v68", "v69", "v70", "v71", "v72", "v73", "v74", "v75", "v76", "v77", "v78", "v79", \
    "v80", "v81", "v82", "v83", "v84", "v85", "v86", "v87", "v88", "v89", "v90", "v91", "v92", "v93", "v94", "v95", \
    "v96", "v97", "v98", "v99", "v100", "v101", "v102", "v103", "v104", "v105", "v106", "v107", "v108", "v109", "v110", "v111", \
    "v112", "v113", "v114", "v115", "v116", "v117", "v118", "v119", "v120", "v121", "v122", "v123", "v124", "v125", "v126", "v127", \
    "v192", "v193", "v194", "v195", "v196", "v197", "v198", "v199", "v200", "v201", "v202", "v203", "v204", "v205", "v206", "v207", \
    "v208", "v209", "v210", "v211", "v212", "v213", "v214", "v215", "v216", "v217", "v218", "v219", "v220", "v221", "v222", "v223", \
    "v246", "v247", "v248", "v249", "v250", "v251"

constexpr int kLseWaves = 4;

__global__ __launch_bounds__(kLseWaves * 64, 2) void k_lse_wide_bf16(AttnArgs a) {
    extern __shared__ __attribute__((aligned(256))) char smem[];
    int c, h, qt, sp;
    if (!work_item(a, c, h, qt, sp)) return;
    const Window win = window_of(a, c);
    const int n_kv = win.n_kv;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int lane = tid & 63, col = lane & 31, g = lane >> 5;
    const int q0 = qt * 256 + wave * 64;   // the wave's first query; a lane has q0 + col and q0 + 32 + col
    float *const out = win.lse + (size_t)h * a.q_rows + a.q_off;
    if (n_kv == 0) {
        if (q0 + lane < a.N_q) out[q0 + lane] = -INFINITY;
        return;
    }
    bf16x8 qb[2][8];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const char *Qrow = a.Q + ((size_t)h * a.q_rows + a.q_off + min(q0 + 32 * q + col, a.N_q - 1)) * 256;
#pragma unroll
        for (int st = 0; st < 8; ++st) qb[q][st] = *reinterpret_cast<const bf16x8 *>(Qrow + (2 * st + g) * 16);
    }
    const unsigned lds0 = (unsigned)(size_t)WK_LDS(smem);
    unsigned k_rd[8];   // as in k_attn_bf16: chunk 2*st + g of key col, slot c ^ (key & 15)
#pragma unroll
    for (int st = 0; st < 8; ++st) k_rd[st] = lds0 + col * 256 + (((2 * st + g) ^ (col & 15)) << 4);
    // tile loads: a wave fills 1 KB blocks 4*wave .. 4*wave + 3 of a tile; rows past the window become its last one
    unsigned k_src[4], k_lim[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int R = 4 * (4 * wave + i) + (lane >> 4);
        k_src[i] = R * 256 + (((lane & 15) ^ (R & 15)) << 4);
        k_lim[i] = (unsigned)(n_kv - 1) * 256u + (k_src[i] & 255u);
    }
    const char *const Kh = uniform_ptr(win.K + (size_t)h * win.stride * 256);
    const unsigned dma_dst = lds0 + wave * 4096;
    auto issue_tile = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const unsigned off = min((unsigned)t * (kKeys * 256u) + k_src[i], k_lim[i]);
            unsigned callers_m0;   // in assembly: the compiler would wait for every load in flight before each operand read
            asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b32 m0, %0"
                         : "=&s"(callers_m0) : "s"(dma_dst + (t & 3) * kTileBytes + i * 1024), "v"(off), "s"(Kh) : "memory");
        }
    };
    auto barrier = [&]() __attribute__((always_inline)) {   // (a bare one: __syncthreads would wait for the loads in flight too)
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };
    const int n_steps = (n_kv + kKeys - 1) / kKeys - 1;   // a step forms S^T of tile j + 1, sums tile j and requests tile j + 4
#pragma unroll
    for (int t = 0; t < 4; ++t) issue_tile(t);
    __builtin_amdgcn_s_waitcnt(0x0F7C);   // vmcnt(12): tile 0
    barrier();
    if (q0 >= a.N_q) {   // no valid query in this wave: its share of the loads and the barriers
        __builtin_amdgcn_s_waitcnt(0x0F78);
        barrier();
        for (int j = 0; j < n_steps; ++j) {
            issue_tile(j + 4);
            __builtin_amdgcn_s_waitcnt(0x0F78);
            barrier();
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);
        return;
    }
    auto from_ring = [&](int kb, int st) __attribute__((always_inline)) { return *WK_LDS_AT(const bf16x8, k_rd[st] + kb * 8192); };
    auto scores = [&](auto &&keys, f32x16 (&s)[2][2]) __attribute__((always_inline)) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int r = 0; r < 16; ++r) s[kb][q][r] = 0.f;
#pragma unroll
            for (int st = 0; st < 8; ++st) {
                const bf16x8 ka = keys(kb, st);
#pragma unroll
                for (int q = 0; q < 2; ++q) s[kb][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qb[q][st], s[kb][q], 0, 0, 0);
            }
        }
    };
    const float c_log2 = a.scale_log2;
    auto tile_max = [&](const f32x16 (&s)[2][2], int q) __attribute__((always_inline)) {
        float m = max3(s[0][q][0], s[0][q][1], s[0][q][2]);
#pragma unroll
        for (int r = 3; r < 31; r += 2) m = max3(m, s[r >> 4][q][r & 15], s[(r + 1) >> 4][q][(r + 1) & 15]);
        return max_across_halves(fmaxf(m, s[1][q][15])) * c_log2;
    };
    float m_run[2];      // reference
    float l_run[2][2];   // row sums [parity of the tile][query block], as in k_attn_bf16
    // (as the loop does it)
    auto sum_tile = [&](f32x16 (&s)[2][2], float (&l)[2], float (&l_other)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const float neg_m = -m_run[q], before = l[q];
            const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int e = 0; e < 16; e += 2) {
                    s[kb][q][e] = __builtin_amdgcn_exp2f(fmaf(s[kb][q][e], c_log2, neg_m));
                    s[kb][q][e + 1] = __builtin_amdgcn_exp2f(fmaf(s[kb][q][e + 1], c_log2, neg_m));
                    l[q] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_convertvector(f32x2{s[kb][q][e], s[kb][q][e + 1]}, bf16x2), ones, l[q], false);
                }
            if (__any(l[q] >= before + 256.0f)) {
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int e = 0; e < 16; e += 2)
                        l[q] += __builtin_amdgcn_fdot2_f32_bf16(__builtin_convertvector(f32x2{s[kb][q][e], s[kb][q][e + 1]}, bf16x2), -ones,
                                                                s[kb][q][e] + s[kb][q][e + 1], false);
                const int own = __builtin_amdgcn_frexp_expf(l[q] - before) - 5, up = max(0, max(own, __shfl_xor(own, 32)));
                m_run[q] += (float)up;
                l[q] = ldexpf(l[q], -up);
                l_other[q] = ldexpf(l_other[q], -up);
            }
        }
    };
    auto swap_parity = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const float t = l_run[0][q];
            l_run[0][q] = l_run[1][q];
            l_run[1][q] = t;
        }
    };
    auto mask_tail = [&](f32x16 (&s)[2][2]) __attribute__((always_inline)) {   // keys past the window (last tile)
        const int kt = n_steps * kKeys;
        if (kt + kKeys <= n_kv) return;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (kt + 32 * kb + 8 * (r >> 2) + 4 * g + (r & 3) >= n_kv) s[kb][0][r] = s[kb][1][r] = -INFINITY;
    };
    f32x16 s_a[2][2];
    scores(from_ring, s_a);
    __builtin_amdgcn_s_waitcnt(0x0F78);   // vmcnt(8): tile 1
    barrier();                            // and tile 0 has been read by every wave
    if (n_steps == 0) mask_tail(s_a);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        m_run[q] = fmaxf(-FLT_MAX, tile_max(s_a, q));
        l_run[0][q] = l_run[1][q] = 0.f;
    }
    if (n_steps > 0) {
        int steps = n_steps - 1;
        unsigned dst = dma_dst;
        // K rows of this head from tile 4 on as a raw buffer, which ends behind the window's last row
        const uint64_t from = reinterpret_cast<uint64_t>(Kh) + 4 * (kKeys * 256u);
        const unsigned bytes = (unsigned)n_kv * 256u, skipped = 4 * (kKeys * 256u);
        const auto scalar = [](unsigned x) { return (unsigned)__builtin_amdgcn_readfirstlane((int)x); };
        u32x4 rows = {scalar((unsigned)from), scalar((unsigned)(from >> 32) & 0xffffu), scalar(bytes > skipped ? bytes - skipped : 0u), scalar(0x00020000u)};
        f32x16 s00 = s_a[0][0], s01 = s_a[0][1], s10 = s_a[1][0], s11 = s_a[1][1];
        // (in and out, so that nothing that the loop leaves alone needs a second register)
        bf16x8 q00 = qb[0][0], q01 = qb[0][1], q02 = qb[0][2], q03 = qb[0][3], q04 = qb[0][4], q05 = qb[0][5], q06 = qb[0][6], q07 = qb[0][7];
        bf16x8 q10 = qb[1][0], q11 = qb[1][1], q12 = qb[1][2], q13 = qb[1][3], q14 = qb[1][4], q15 = qb[1][5], q16 = qb[1][6], q17 = qb[1][7];
        unsigned r0 = k_rd[0], r1 = k_rd[1], r2 = k_rd[2], r3 = k_rd[3], r4 = k_rd[4], r5 = k_rd[5], r6 = k_rd[6], r7 = k_rd[7];
        asm volatile(
#include "wk_lse_loop_gfx950.inc"
            : "+{v[0:15]}"(s00), "+{v[16:31]}"(s01), "+{v[32:47]}"(s10), "+{v[48:63]}"(s11), "+{v240}"(m_run[0]), "+{v241}"(m_run[1]),
              "+{v242}"(l_run[0][0]), "+{v243}"(l_run[0][1]), "+{v244}"(l_run[1][0]), "+{v245}"(l_run[1][1]),
              "+{v224}"(r0), "+{v225}"(r1), "+{v226}"(r2), "+{v227}"(r3), "+{v228}"(r4), "+{v229}"(r5), "+{v230}"(r6), "+{v231}"(r7),
              "+{v[128:131]}"(q00), "+{v[132:135]}"(q01), "+{v[136:139]}"(q02), "+{v[140:143]}"(q03), "+{v[144:147]}"(q04), "+{v[148:151]}"(q05),
              "+{v[152:155]}"(q06), "+{v[156:159]}"(q07), "+{v[160:163]}"(q10), "+{v[164:167]}"(q11), "+{v[168:171]}"(q12), "+{v[172:175]}"(q13),
              "+{v[176:179]}"(q14), "+{v[180:183]}"(q15), "+{v[184:187]}"(q16), "+{v[188:191]}"(q17), "+{v232}"(k_src[0]), "+{v233}"(k_src[1]),
              "+{v234}"(k_src[2]), "+{v235}"(k_src[3]), "+{s[36:39]}"(rows), "+{s42}"(dst), "+{s44}"(steps)
            : "{s43}"(c_log2)
            : WK_LSE_LOOP_CLOBBERS, "s45", "s46", "s47", "s48", "s49", "vcc", "memory");
        s_a[0][0] = s00; s_a[0][1] = s01; s_a[1][0] = s10; s_a[1][1] = s11;
        qb[0][0] = q00; qb[0][1] = q01; qb[0][2] = q02; qb[0][3] = q03; qb[0][4] = q04; qb[0][5] = q05; qb[0][6] = q06; qb[0][7] = q07;
        qb[1][0] = q10; qb[1][1] = q11; qb[1][2] = q12; qb[1][3] = q13; qb[1][4] = q14; qb[1][5] = q15; qb[1][6] = q16; qb[1][7] = q17;
        // (known anew, so that nothing made of them waits in scratch while the loop has the registers)
        asm("" : "+v"(lane));
        col = lane & 31, g = lane >> 5;
        mask_tail(s_a);   // the last tile: the only one that can be partial
    }
    if (n_steps & 1) swap_parity();
    sum_tile(s_a, l_run[0], l_run[1]);
    __builtin_amdgcn_s_waitcnt(0x0F70);   // the clamped look-ahead loads have landed
    // Scores that exceed the reference by 2^126 within a tile: such a wave starts again by itself, with a running maximum and its
    // operands straight from global memory.
    const bool sum_fits = (__float_as_uint(l_run[0][0] + l_run[1][0]) & 0x7fffffffu) < 0x7e800000u &&
                          (__float_as_uint(l_run[0][1] + l_run[1][1]) & 0x7fffffffu) < 0x7e800000u;   // (nor is it a NaN)
    if (__any(!sum_fits)) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            m_run[q] = -FLT_MAX;
            l_run[0][q] = l_run[1][q] = 0.f;
        }
        for (int t = 0; t <= n_steps; ++t) {
            scores([&](int kb, int st) __attribute__((always_inline)) {
                const size_t row = min(t * kKeys + 32 * kb + col, n_kv - 1);
                return *reinterpret_cast<const bf16x8 *>(Kh + row * 256 + (2 * st + g) * 16);
            }, s_a);
            if (t == n_steps) mask_tail(s_a);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const float m_new = fmaxf(m_run[q], tile_max(s_a, q)), alpha = __builtin_amdgcn_exp2f(m_run[q] - m_new);
                l_run[0][q] *= alpha;
                l_run[1][q] *= alpha;
                m_run[q] = m_new;
            }
            sum_tile(s_a, l_run[0], l_run[1]);
            swap_parity();
        }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const float l_lane = l_run[0][q] + l_run[1][q];
        const float l_tot = l_lane + __shfl_xor(l_lane, 32);
        const int query = q0 + 32 * q + col;
        if (query < a.N_q && g == 0) out[query] = (m_run[q] + log2f(l_tot)) * 0.6931471805599453f;
    }
}

// Bound by its reads of the partial results (516 bytes per row and split), with the loads of four splits in flight: 6 us
// for 9 splits of 3,520 rows, where one split at a time took 9 us.
// Merge of the key-range splits: O = sum_s 2^(m_s - m) O_s / sum_s 2^(m_s - m) l_s, m = max_s m_s.
// 16 lanes per query row, 8 features each; fixed summation order.
template <int DT>
__global__ __launch_bounds__(256) void k_attn_merge(AttnArgs a) {
    const size_t row = (size_t)blockIdx.x * 16 + threadIdx.x / 16;   // h * q_rows + q
    const int sub = threadIdx.x % 16;
    const size_t rows = (size_t)a.H * a.q_rows;
    if (row >= rows) return;
    // four splits' loads are in flight at a time (a split past the last one repeats its loads and is left out of the sums, as
    // is a split with no weight at all: an infinity or NaN times a weight of zero would not be zero)
    constexpr int kBatch = 4;
    const float2 *ml = reinterpret_cast<const float2 *>(a.part_ml) + row;
    float m = -INFINITY;
    for (int s0 = 0; s0 < a.splits; s0 += kBatch) {
        float ms[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) ms[u] = ml[min(s0 + u, a.splits - 1) * rows].x;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) m = fmaxf(m, ms[u]);
    }
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    float l = 0.f;
    for (int s0 = 0; s0 < a.splits; s0 += kBatch) {
        float2 t[kBatch];
        float4 x[kBatch], y[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const size_t at = min(s0 + u, a.splits - 1) * rows;
            t[u] = ml[at];
            const float4 *po = reinterpret_cast<const float4 *>(a.part_o + (at + row) * WK_D) + 2 * sub;
            x[u] = po[0];
            y[u] = po[1];
        }
        asm volatile("" ::: "memory");   // the loads stay together, in front of the branches
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            if (s0 + u >= a.splits || t[u].x == -INFINITY) continue;
            const float w = __builtin_amdgcn_exp2f(t[u].x - m);
            l = fmaf(w, t[u].y, l);
            acc[0] = fmaf(w, x[u].x, acc[0]); acc[1] = fmaf(w, x[u].y, acc[1]); acc[2] = fmaf(w, x[u].z, acc[2]); acc[3] = fmaf(w, x[u].w, acc[3]);
            acc[4] = fmaf(w, y[u].x, acc[4]); acc[5] = fmaf(w, y[u].y, acc[5]); acc[6] = fmaf(w, y[u].z, acc[6]); acc[7] = fmaf(w, y[u].w, acc[7]);
        }
    }
    const float inv = l > 0.f ? 1.f / l : 0.f;
    if constexpr (DT == WK_BF16) {
        uint4 out;
        uint32_t *ow = reinterpret_cast<uint32_t *>(&out);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            ow[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{acc[2 * e] * inv, acc[2 * e + 1] * inv}, bf16x2));
        reinterpret_cast<uint4 *>(a.O + row * 256)[sub] = out;
    } else {
        float4 *po = reinterpret_cast<float4 *>(a.O + row * 512) + 2 * sub;
        po[0] = float4{acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv};
        po[1] = float4{acc[4] * inv, acc[5] * inv, acc[6] * inv, acc[7] * inv};
    }
    if (a.lse && sub == 0) a.lse[row] = l > 0.f ? (m + log2f(l)) * 0.6931471805599453f : -INFINITY;
}

// How a bf16 launch is laid out:
//   k256      workgroups of 256 queries, a tile of 64 keys per step
//   k128Pair  workgroups of 128 queries, a pair of tiles per step: twice the workgroups, 10 % more power per product
//             (every tile is fetched for half as many queries)
//   k128      workgroups of 128 queries in four waves, a tile per step: no pair to wait for, no wave groups to meet
//   splits    > 1: the key range split over workgroups and merged (needs a workspace), at most kMaxSplits and a step or
//             more of work each
// chosen by the cheapest predicted time.  A step takes longer with more compute units at work, because the chip lowers
// its clock: busy_us with few of them, full_us with all 256; a workgroup's fill and drain cost fill_steps; a launch has
// launch_us of its own, whatever its size (a pair's meeting among it); the merge a launch, its traffic and a round trip for
// every four splits.  The figures were fitted to timed launches of 851 shapes (2 to 40 heads, 64 to 4,680 queries, 64 to
// 211,200 keys, with and without a workspace, inputs in turn) in all layouts and split counts: over those the rule's choice is
// 0.4 % slower than the fastest on average, 10 % at most, and never more than 4 % slower than the choice between k256 with splits
// and k128 that went before k128Pair.
// k128 is the best for up to 5 tiles and for 7 and 9 (an odd count leaves one wave group of a pair idle for a step): 12 heads x 512
// queries x 64 keys 6.9 us, in pairs 8.9 us, x 448 13.0 and 13.7 us; x 768 17.4 and 17.0 us.
// Predictions of one layout within 0.3 % count as equal and the fewer splits are taken: 12 heads x 2,640 queries x 211,200 keys take 3.0 ms
// with 11, 13 and 15 splits alike.
// (Query tiles that walk the same slice of a head's keys run side by side and share it through the L2, which cutting the
// work into equal runs regardless of item boundaries would give up: that was measured 5 to 14 % slower.)
enum Layout { k256, k128Pair, k128, kLayouts };
constexpr int kMaxSplits = 16;
constexpr int kMinSplitTiles = 24;   // shorter windows: a workspace would buy less than 2 us

size_t split_workspace_bytes(int H, int N_q, int splits) {
    const size_t rows = (size_t)splits * H * N_q;
    return wk::align_up(rows * WK_D * sizeof(float), 256) + wk::align_up(rows * 2 * sizeof(float), 256);
}

struct LayoutModel { int qw, kg; double busy_us, full_us, fill_steps, launch_us; };
constexpr LayoutModel kModel[kLayouts] = {{8, 1, 1.22, 1.35, 1.2, 5.8}, {4, 2, 1.47, 1.67, 1.2, 6.0}, {4, 1, 1.01, 1.04, 5.8, 0.0}};

struct LaunchPlan { Layout layout; int splits; };

constexpr int queries_per_wg(Layout l) { return 32 * kModel[l].qw; }

// wgs workgroups of `steps` steps each (on average)
double grid_us(const LayoutModel &m, long long wgs, double steps) {
    const double rest = (double)(wgs % 256) / 256;
    return m.launch_us + (steps + m.fill_steps) * ((double)(wgs / 256) * m.full_us + (rest == 0 ? 0 : std::fmax(m.busy_us, m.full_us * rest)));
}

// the partial results' way to memory and back, and the merge
double merge_us(int splits, long long rows) { return 2.0 + 0.86 * ((splits + 3) / 4) + 2.0 * splits * (double)rows * 516.0 / 5.1e6; }

double launch_us(Layout l, int splits, long long H, long long N_q, int n_tiles) {
    const LayoutModel &m = kModel[l];
    const long long wgs = H * ((N_q + queries_per_wg(l) - 1) / queries_per_wg(l)) * splits;
    const int tiles = (n_tiles + splits - 1) / splits, steps = (tiles + m.kg - 1) / m.kg;
    double us = grid_us(m, wgs, steps);
    if (splits > 1) us += merge_us(splits, H * N_q);
    return us;
}

// the best plan whose partial results fit workspace_bytes
LaunchPlan plan_bf16(int H, int N_q, int N_kv, size_t workspace_bytes) {
    const int n_tiles = (N_kv + 63) / 64;
    LaunchPlan best{k256, 1};
    double best_us = launch_us(k256, 1, H, N_q, n_tiles);
    for (const Layout l : {k256, k128Pair, k128}) {
        for (int sp = 1; sp <= (l == k128 ? 1 : kMaxSplits); ++sp) {
            if (sp > 1 && (n_tiles < std::max(2 * kModel[l].kg * sp, kMinSplitTiles) || split_workspace_bytes(H, N_q, sp) > workspace_bytes)) break;
            const double us = launch_us(l, sp, H, N_q, n_tiles);
            if (us < (l == best.layout ? 0.997 : 1.0) * best_us) {
                best_us = us;
                best = LaunchPlan{l, sp};
            }
        }
    }
    return best;
}

// The workgroup size of a table of launches, by the same model: the grid's time if every workgroup had the average
// number of steps, or the longest workgroup's alone.
Layout table_layout(const SubTable &t, long long H, double &best_us) {
    Layout best = k256;
    for (const Layout l : {k256, k128Pair}) {
        const LayoutModel &m = kModel[l];
        long long wgs = 0, steps = 0, longest = 0;
        for (int e = 0; e < t.n; ++e) {
            const long long n = H * ((t.s[e].N_q + queries_per_wg(l) - 1) / queries_per_wg(l)), tiles = (t.s[e].N_kv - t.s[e].gap_len + 63) / 64;
            const long long len = (tiles + m.kg - 1) / m.kg;
            wgs += n;
            steps += n * len;
            longest = std::max(longest, len);
        }
        const double us = std::fmax(grid_us(m, wgs, (double)steps / (double)wgs), grid_us(m, std::min(wgs, 256ll), (double)longest));
        if (l == k256 || us < best_us) {
            best = l;
            best_us = us;
        }
    }
    return best;
}

// The visible key ranges of a frame-masked call as launches: entry 0 = the rows behind the chunk for every query (the long items
// first), entries 1.. = the prefix up to frame f for that frame's queries.
SubTable frame_table(int N_q, int N_kv, int row0, int frame_T) {
    SubTable t{};
    t.n = N_q / frame_T + 1;
    const int start = row0 + N_q;
    t.s[0] = SubLaunch{0, N_q, 0, start, N_kv - start, start, 1, 0, 0};
    for (int f = 0; f + 1 < t.n; ++f) t.s[f + 1] = SubLaunch{f * frame_T, frame_T, 0, 0, row0 + (f + 1) * frame_T, 0, 0, 0, 0};
    return t;
}

// The same call with one entry per frame, whose window leaves out the later frames of the chunk: no partial results, no merge.
SubTable frame_gap_table(int N_q, int N_kv, int row0, int frame_T) {
    SubTable t{};
    t.n = N_q / frame_T;
    for (int e = 0; e < t.n; ++e) {   // the longest first
        const int f = t.n - 1 - e;
        t.s[e] = SubLaunch{f * frame_T, frame_T, 0, 0, N_kv, 0, -1, row0 + (f + 1) * frame_T, e * frame_T};
    }
    return t;
}

// Windows with a gap where the model prefers them: a query's keys are walked once, by one workgroup, where the two ranges begin and
// end two, write their partial results and merge them.  12 heads x 3 frames of 880 queries on 10,560 keys: 252 workgroups of 128
// queries 160 us; two ranges, 504 workgroups and a merge, 175 us.  17 x 3 x 558 on 4,464 keys 92 -> 69 us, 48 x 3 x 300 on
// 900 58 -> 36, 2 x 3 x 250 on 750 19.7 -> 16.7.  Two ranges where the frames alone leave compute units idle, as splits of the keys:
// 5 heads x 2 x 993 on 8,440 keys 75 us, with a gap 103; 40 x 3 x 1,560 on 28,080 keys 2,292 and 2,372.
// Over 1,500 drawn shapes (2 to 64 heads, 1 to 7 frames of 16 to 1,560 queries, both forms in both workgroup sizes timed) the choice is 10 % faster
// than two ranges alone and 0.8 % slower than the best, on average; it is more than 2 % slower than two ranges alone on 17, by 12 % at most:
// the model takes a last, partly filled round for a whole one, also where workgroups of unequal length fill it (8 x 2 x 1,231 on 9,848 keys:
// 122 us, two ranges 109; and 40 x 3 x 1,560 on 14,040: two ranges 1,167, windows with a gap in 256-query workgroups 1,118).
struct FramePlan { SubTable table; Layout layout; bool merge; };

FramePlan plan_frames(int H, int N_q, int N_kv, int row0, int frame_T) {
    double us = 0, gap_us = 0;
    FramePlan p{frame_table(N_q, N_kv, row0, frame_T), k256, true}, g{frame_gap_table(N_q, N_kv, row0, frame_T), k256, false};
    p.layout = table_layout(p.table, H, us);
    g.layout = table_layout(g.table, H, gap_us);
    us += merge_us(2, (long long)H * N_q);
    return gap_us < us ? g : p;
}

// fp32: the wave groups (KG) and key ranges with the cheapest predicted time.  A step of one workgroup per compute unit takes 1.9 us with one tile at a
// time; of two workgroups per unit 2.6, and 3.0 once all 256 have two; with two tiles at a time 3.0 (3.2 on all units) and a step's time for
// the groups to meet; a call 11 us beside its steps and its merge.  Fitted to 12 shapes (1 to 40 heads, 128 to 4,000 queries, 100 to 9,000 keys) in
// every form and count of ranges: 5 % off (rms), and the choice 0.3 % slower than the best.  4 heads x 880 queries x 2,640 keys in two groups and 9
// ranges 39 us, in one group and 8 ranges 41, in one range 139 and 180; 40 x 1,560 x 4,680 in one group and 5 ranges 589 us, in 2 ranges
// 633, in one 750 (520 workgroups are two rounds of 512).
// Ranges of two steps and more, and none below 8 tiles, where the order of sums would depend on the host's bound of a length that
// the device knows; nor do the groups of an undivided window depend on it beyond the first tile, whose sums are the same in one and in two.
struct F32Plan { int kg, splits; };

double f32_step_us(int kg, long long wgs) {   // of up to 512 / kg workgroups
    if (kg == 2) return wgs > 224 ? 3.2 : 3.0;
    return wgs <= 256 ? 1.9 : 2.6 + 0.4 * (double)(wgs - 256) / 256;
}

F32Plan plan_f32(long long H, long long N_q, int n_tiles, size_t workspace_bytes) {
    const long long items = H * ((N_q + kF32Waves * 32 - 1) / (kF32Waves * 32));
    const int whole = n_tiles > 1 && items <= 256 ? 2 : 1;   // wave groups of an undivided window
    F32Plan best{whole, 1};
    double best_us = 0;
    for (const int kg : {whole, 3 - whole}) {
        const long long slots = 512 / kg;
        for (int s = kg == whole ? 1 : 2; s <= kMaxSplits; ++s) {
            if (s > 1 && (n_tiles < std::max(8, 2 * kg * s) || split_workspace_bytes((int)H, (int)N_q, s) > workspace_bytes)) break;
            const int steps = ((n_tiles + s - 1) / s + kg - 1) / kg + (kg - 1);
            const long long wgs = items * s, rest = wgs % slots;
            double us = steps * ((double)(wgs / slots) * f32_step_us(kg, slots) + (rest ? f32_step_us(kg, rest) : 0.0));
            if (s > 1) us += merge_us(s, H * N_q);
            if (best_us == 0 || us < best_us) {
                best = F32Plan{kg, s};
                best_us = us;
            }
        }
    }
    return best;
}

// k_attn_bf16 and k_attn_f32 use more than the default 64 KB of dynamic LDS: raise its limit once per device and
// process (not a stream operation, so a first call under graph capture is fine too).
wk_status allow_large_lds() {
    static std::atomic<uint64_t> done{0};
    int dev;
    if (wk::device_needs_setup(done, dev)) {
        struct { const void *kernel; int bytes; } const kernels[] = {
            {reinterpret_cast<const void *>(&k_attn_bf16<8, 1, false, false>), kSmemBytes},
            {reinterpret_cast<const void *>(&k_attn_bf16<8, 1, true, false>), kSmemBytes},
            {reinterpret_cast<const void *>(&k_attn_bf16<8, 1, true, false, true>), kSmemBytes},
            {reinterpret_cast<const void *>(&k_attn_bf16<8, 1, false, true>), kSmemBytes},
            {reinterpret_cast<const void *>(&k_attn_bf16<8, 1, false, true, false, true>), kSmemBytes},
            {reinterpret_cast<const void *>(&k_attn_bf16<4, 2, false, false>), kSmemBytes},
            {reinterpret_cast<const void *>(&k_attn_bf16<4, 2, true, false>), kSmemBytes},
            {reinterpret_cast<const void *>(&k_attn_bf16<4, 2, true, false, true>), kSmemBytes},
            {reinterpret_cast<const void *>(&k_attn_bf16<4, 2, false, true>), kSmemBytes},
            {reinterpret_cast<const void *>(&k_attn_bf16<4, 2, false, true, false, true>), kSmemBytes},
            {reinterpret_cast<const void *>(&k_attn_bf16<4, 1, false, false>), kSmemBytes},
            {reinterpret_cast<const void *>(&k_attn_bf16<4, 1, false, true>), kSmemBytes},
            {reinterpret_cast<const void *>(&k_attn_f32<1, false, true>), kF32Lds},
            {reinterpret_cast<const void *>(&k_attn_f32<1, true, true>), kF32Lds},
            {reinterpret_cast<const void *>(&k_attn_f32<1, false, false>), kF32Lds},
            {reinterpret_cast<const void *>(&k_attn_f32<2, false, false>), kF32LdsPair},
            {reinterpret_cast<const void *>(&k_attn_f32<2, false, true>), kF32LdsPair},
            {reinterpret_cast<const void *>(&k_attn_f32<2, true, true>), kF32LdsPair},
        };
        for (const auto &k : kernels)
            if (hipFuncSetAttribute(k.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, k.bytes) != hipSuccess) return WK_ERR_HIP;
        wk::mark_device(done, dev);
    }
    return WK_OK;
}

// k_lse_wide_bf16 where windows are long enough for its loop to matter and its four waves have queries: 8 chunks of 1,560 keys x 40
// heads x 256 queries 55.2 -> 48.1 us, 24 of 640 x 8 x 877 36.9 -> 33.9, one of 641 x 16 x 1,000 15.8 -> 14.8; but one of 601 x 8 x 877 15.6 -> 16.6,
// 117 of 597 x 8 x 143 43.7 -> 47.5.  A store's lengths lie on the device, and the host goes by its bound, max_tok: chunks that are much
// shorter gain nothing (60 of 256 keys x 12 x 2,640 154 -> 148 us, 24 x 8 x 877 18.0 -> 18.0), and lose up to 4 % where they are few
// (8 of 256 x 40 x 256 13.6 -> 14.1); one long chunk in eight outweighs that (51.4 -> 43.8).
bool lse_wide(const AttnArgs &a) { return (a.n_chunks > 0 ? a.max_tok : a.N_kv) > 10 * kKeys && a.N_q > 192; }

// In place: whether most tiles lie deep enough in their segments for the hand-scheduled loop, which begins once the tiles ahead are of one segment and
// ends before they leave it: about eight tiles of a segment stay outside, in steps that its registers make 4 % slower.
// Without it and with it, by the share of tiles inside: 0.19 (12 heads x 2,640 queries, 12 chunks of 640 keys) 130 and 135 us, 0.38 (of 800) 161 and 164, 0.46 (of
// 900) 180 and 181, 0.55 (of 1,100) 214 and 215, 0.61 (of 1,300) 253 and 252, 0.54 (40 x 2,000, 6 of 900 and 2,000 native) 345 and 343, 0.56 (8 x 900, 8 of 1,200)
// 142 and 135, 0.71 (4 x 300, 3,000 native, 2 of 200) 53 and 49, 0.78 (16 x 3,333, 6,101 native, 7 of 1,747) 470 and 458, 40 x 4,680, 9,360 native, 8 of 2,340
// 2,311 and 2,247.
bool trips_in_place(long long n_native, long long R, long long max_tok) {
    const long long native = (n_native + kKeys - 1) / kKeys, chunk = (max_tok + kKeys - 1) / kKeys;
    return 100 * (std::max(native - 8, 0ll) + R * std::max(chunk - 8, 0ll)) >= 55 * (native + R * chunk);
}

template <int QW, int KG, bool MULTI, bool IN_PLACE, bool GAP = false, bool TRIPS = !IN_PLACE>
void launch_layout(const AttnArgs &a, const SubTable &t, hipStream_t st) {
    hipLaunchKernelGGL((k_attn_bf16<QW, KG, MULTI, IN_PLACE, GAP, TRIPS>), dim3(a.per_xcd * kXcds), dim3(QW * KG * 64),
                       kSmemBytes, st, a, t);
}

void partials_in(AttnArgs &a, void *workspace) {   // (O, then maximum and sum) of a.splits key ranges
    a.part_o = reinterpret_cast<float *>(workspace);
    a.part_ml = reinterpret_cast<float *>(reinterpret_cast<char *>(workspace) +
                                          wk::align_up((size_t)a.splits * a.H * a.N_q * WK_D * sizeof(float), 256));
}

template <bool MULTI, bool WITH_O>
void launch_f32_grid(const AttnArgs &a, const SubTable &t, int kg, hipStream_t st) {
    const dim3 grid(a.per_xcd * kXcds);
    if (kg == 2) hipLaunchKernelGGL((k_attn_f32<2, MULTI, WITH_O>), grid, dim3(2 * kF32Waves * 64), kF32LdsPair, st, a, t);
    else hipLaunchKernelGGL((k_attn_f32<1, MULTI, WITH_O>), grid, dim3(kF32Waves * 64), kF32Lds, st, a, t);
}

wk_status launch_f32(AttnArgs a, int kg, hipStream_t st) {
    a.n_qtiles = (a.N_q + kF32Waves * 32 - 1) / (kF32Waves * 32);
    const long long items = (long long)a.H * a.n_qtiles * a.splits * (a.n_chunks > 0 ? a.n_chunks : 1);
    if (!wk::fits_launch(items + kXcds, 2 * kF32Waves * 64)) return WK_ERR_UNSUPPORTED;
    a.per_xcd = (int)((items + kXcds - 1) / kXcds);
    const wk_status rc = allow_large_lds();
    if (rc != WK_OK) return rc;
    if (a.O) launch_f32_grid<false, true>(a, SubTable{}, kg, st);
    else launch_f32_grid<false, false>(a, SubTable{}, kg, st);
    WK_LAUNCH_CHECK();
    return WK_OK;
}

wk_status launch_bf16(AttnArgs a, LaunchPlan plan, void *workspace, hipStream_t st) {
    const int q_per_wg = queries_per_wg(plan.layout);
    a.n_qtiles = (a.N_q + q_per_wg - 1) / q_per_wg;
    a.splits = plan.splits;
    if (a.splits > 1) partials_in(a, workspace);
    const long long items = (long long)a.H * a.n_qtiles * a.splits * (a.n_chunks > 0 ? a.n_chunks : 1);
    const bool wide = !a.O && lse_wide(a);
    if (!wk::fits_launch(items + kXcds, wide ? kLseWaves * 64 : kModel[plan.layout].qw * kModel[plan.layout].kg * 64)) return WK_ERR_UNSUPPORTED;
    a.per_xcd = (int)((items + kXcds - 1) / kXcds);
    const wk_status lds_rc = allow_large_lds();
    if (lds_rc != WK_OK) return lds_rc;
    if (!a.O) {
        if (plan.layout != k256) return WK_ERR_UNSUPPORTED;   // the log-sum-exp kernel is laid out for 256-query workgroups
        if (wide) hipLaunchKernelGGL(k_lse_wide_bf16, dim3(a.per_xcd * kXcds), dim3(kLseWaves * 64), kVRing, st, a);
        else hipLaunchKernelGGL(k_lse_bf16, dim3(a.per_xcd * kXcds), dim3(512), kVRing, st, a);
    } else if (plan.layout == k256) {
        launch_layout<8, 1, false, false>(a, SubTable{}, st);
    } else if (plan.layout == k128Pair) {
        launch_layout<4, 2, false, false>(a, SubTable{}, st);
    } else {
        launch_layout<4, 1, false, false>(a, SubTable{}, st);
    }
    WK_LAUNCH_CHECK();
    if (a.splits > 1) {
        const size_t rows = (size_t)a.H * a.N_q;
        hipLaunchKernelGGL(k_attn_merge<WK_BF16>, dim3((unsigned)((rows + 15) / 16)), dim3(256), 0, st, a);
        WK_LAUNCH_CHECK();
    }
    return WK_OK;
}

}  // namespace

extern "C" wk_status wk_attention(const void *Q, const void *K_win, const void *V_win, void *O, float *lse,
                                  int32_t H, int32_t N_q, int32_t N_kv, int32_t d, int32_t kv_row_stride,
                                  int32_t dtype, float scale, const int32_t *n_kv_dev, void *workspace,
                                  size_t workspace_bytes, void *hip_stream) {
    if (!Q || !K_win) return WK_ERR_INVALID_ARG;
    if (O ? !V_win : !lse) return WK_ERR_INVALID_ARG;   // O == NULL: log-sum-exp only, V is not read
    if (H < 1 || N_q < 0 || d < 1) return WK_ERR_INVALID_ARG;
    if (dtype != WK_F32 && dtype != WK_BF16) return WK_ERR_INVALID_ARG;
    if (!(scale >= 0.f) || std::isinf(scale)) return WK_ERR_INVALID_ARG;
    if (d != WK_D) return WK_ERR_UNSUPPORTED;
    if (N_kv < 1 || N_kv > kv_row_stride) return WK_ERR_SHAPE;
    if (dtype == WK_BF16 && N_kv > kMaxRowsBf16) return WK_ERR_UNSUPPORTED;   // 32-bit byte offsets inside a head
    if (N_q == 0) return WK_OK;
    if ((long long)H * ((N_q + 31) / 32) > 0x7fffffffLL / kMaxSplits) return WK_ERR_UNSUPPORTED;   // grid size
    AttnArgs a;
    a.Q = reinterpret_cast<const char *>(Q);
    a.K = reinterpret_cast<const char *>(K_win);
    a.V = reinterpret_cast<const char *>(V_win);
    a.O = reinterpret_cast<char *>(O);
    a.lse = lse;
    a.H = H; a.N_q = N_q; a.N_kv = N_kv; a.kv_row_stride = kv_row_stride;
    const float sc = scale == 0.f ? 1.f / std::sqrt((float)d) : scale;
    a.scale_log2 = sc * 1.4426950408889634f;
    a.n_kv_dev = n_kv_dev;
    a.splits = 1;
    a.part_o = nullptr;
    a.part_ml = nullptr;
    a.k_table = nullptr;
    a.n_tok = nullptr;
    a.n_chunks = 0;
    a.q_rows = N_q; a.q_off = 0; a.kv_start = 0; a.part_slot = -1;
    a.v_table = nullptr; a.ids = nullptr; a.n_ids = nullptr; a.R_max = 0; a.store_M = 0; a.max_tok = 0;
    const size_t usable_bytes = workspace && reinterpret_cast<uintptr_t>(workspace) % 256 == 0 ? workspace_bytes : 0;
    hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
    if (dtype == WK_F32) {
        const F32Plan plan = plan_f32(H, N_q, (N_kv + kF32Keys - 1) / kF32Keys, O ? usable_bytes : 0);
        a.splits = plan.splits;
        if (a.splits > 1) partials_in(a, workspace);
        const wk_status rc = launch_f32(a, plan.kg, st);
        if (rc != WK_OK) return rc;
        if (a.splits > 1) {
            const size_t rows = (size_t)H * N_q;
            hipLaunchKernelGGL(k_attn_merge<WK_F32>, dim3((unsigned)((rows + 15) / 16)), dim3(256), 0, st, a);
            WK_LAUNCH_CHECK();
        }
        return WK_OK;
    }
    if (!O) return launch_bf16(a, LaunchPlan{k256, 1}, nullptr, st);   // log-sum-exp only
    return launch_bf16(a, plan_bf16(H, N_q, N_kv, usable_bytes), workspace, st);
}

namespace {

// One launch of the attention kernel for the dtype, exactly as the arguments say: no choice of
// key-range splits, no merge.
wk_status launch_plain(AttnArgs a, int dtype, hipStream_t st) {
    a.splits = 1;
    if (dtype == WK_F32) return launch_f32(a, plan_f32(a.H, a.N_q, (a.N_kv + kF32Keys - 1) / kF32Keys, 0).kg, st);
    a.n_qtiles = (a.N_q + 255) / 256;
    if (!wk::fits_launch((long long)a.H * a.n_qtiles + kXcds, 512)) return WK_ERR_UNSUPPORTED;
    a.per_xcd = (a.H * a.n_qtiles + kXcds - 1) / kXcds;
    const wk_status rc = allow_large_lds();
    if (rc != WK_OK) return rc;
    launch_layout<8, 1, false, false>(a, SubTable{}, st);
    WK_LAUNCH_CHECK();
    return WK_OK;
}

}  // namespace

extern "C" size_t wk_attention_block_causal_workspace_bytes(int32_t H, int32_t N_q) {
    if (H < 1 || N_q < 1) return 0;
    return split_workspace_bytes(H, N_q, 2);
}

// Frame-level causal mask inside the chunk being denoised.  A frame's queries (they share their keys) either attend the window with
// the chunk's later frames left out, or two key ranges whose partial (O, max, sum) results k_attn_merge combines: range A =
// window rows up to and including their own frame of the chunk, range B = the rows behind the chunk (shared by all queries); fp32
// always the latter.  A workgroup is only told which queries, which rows and which partial slot are its own -- through a table of
// up to 8 such entries served by one grid, or, where two ranges need more entries than that, by one launch per entry.
extern "C" wk_status wk_attention_block_causal(const void *Q, const void *K_win, const void *V_win, void *O,
                                               float *lse, int32_t H, int32_t N_q, int32_t N_kv, int32_t d,
                                               int32_t kv_row_stride, int32_t dtype, float scale,
                                               const int32_t *n_kv_dev, int32_t denoise_row0, int32_t frame_T,
                                               void *workspace, size_t workspace_bytes, void *hip_stream) {
    if (!Q || !K_win || !V_win || !O) return WK_ERR_INVALID_ARG;
    if (H < 1 || N_q < 0 || d < 1 || frame_T < 1 || denoise_row0 < 0) return WK_ERR_INVALID_ARG;
    if (dtype != WK_F32 && dtype != WK_BF16) return WK_ERR_INVALID_ARG;
    if (!(scale >= 0.f) || std::isinf(scale)) return WK_ERR_INVALID_ARG;
    if (d != WK_D) return WK_ERR_UNSUPPORTED;
    if (N_kv < 1 || N_kv > kv_row_stride) return WK_ERR_SHAPE;
    if (N_q % frame_T != 0 || (int64_t)denoise_row0 + N_q > (int64_t)N_kv) return WK_ERR_SHAPE;
    if (dtype == WK_BF16 && N_kv > kMaxRowsBf16) return WK_ERR_UNSUPPORTED;   // 32-bit byte offsets inside a head
    if (N_q == 0) return WK_OK;
    if (!workspace || workspace_bytes < split_workspace_bytes(H, N_q, 2) ||
        reinterpret_cast<uintptr_t>(workspace) % 256 != 0)
        return WK_ERR_WORKSPACE;
    const size_t row_bytes = WK_D * wk::esize(dtype);
    AttnArgs a;
    a.Q = reinterpret_cast<const char *>(Q);
    a.K = reinterpret_cast<const char *>(K_win);
    a.V = reinterpret_cast<const char *>(V_win);
    a.O = reinterpret_cast<char *>(O);
    a.lse = lse;
    a.H = H; a.N_q = N_q; a.N_kv = N_kv; a.kv_row_stride = kv_row_stride;
    const float sc = scale == 0.f ? 1.f / std::sqrt((float)d) : scale;
    a.scale_log2 = sc * 1.4426950408889634f;
    a.n_kv_dev = n_kv_dev;
    a.splits = 1;
    a.part_o = reinterpret_cast<float *>(workspace);
    a.part_ml = reinterpret_cast<float *>(reinterpret_cast<char *>(workspace) +
                                          wk::align_up((size_t)2 * H * N_q * WK_D * sizeof(float), 256));
    a.k_table = nullptr; a.n_tok = nullptr; a.n_chunks = 0;
    a.q_rows = N_q; a.q_off = 0; a.kv_start = 0; a.part_slot = -1;
    a.v_table = nullptr; a.ids = nullptr; a.n_ids = nullptr; a.R_max = 0; a.store_M = 0; a.max_tok = 0;
    hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);

    const int frames = N_q / frame_T;
    const int start = denoise_row0 + N_q;
    if (frames + 1 <= kMaxSub) {
        FramePlan plan;   // all ranges in one grid
        if (dtype == WK_F32) plan = FramePlan{frame_table(N_q, N_kv, denoise_row0, frame_T), k256, true};   // (fp32 has a layout of its own)
        else plan = plan_frames(H, N_q, N_kv, denoise_row0, frame_T);
        SubTable &t = plan.table;
        const Layout layout = plan.layout;
        const int q_per_wg = dtype == WK_F32 ? kF32Waves * 32 : queries_per_wg(layout);
        t.per_head = 0;
        for (int e = 0; e < t.n; ++e) {
            t.s[e].n_qtiles = (t.s[e].N_q + q_per_wg - 1) / q_per_wg;
            t.per_head += t.s[e].n_qtiles;
        }
        AttnArgs g = a;
        if (!wk::fits_launch((long long)H * t.per_head + kXcds, 512)) return WK_ERR_UNSUPPORTED;
        g.per_xcd = (H * t.per_head + kXcds - 1) / kXcds;
        g.n_qtiles = 0;
        const wk_status lrc = allow_large_lds();
        if (lrc != WK_OK) return lrc;
        if (dtype == WK_F32) {
            launch_f32_grid<true, true>(g, t, plan_f32(1, (long long)H * t.per_head * kF32Waves * 32, (N_kv + kF32Keys - 1) / kF32Keys, 0).kg, st);
        } else {
            if (layout == k256 && !plan.merge) launch_layout<8, 1, true, false, true>(g, t, st);
            else if (!plan.merge) launch_layout<4, 2, true, false, true>(g, t, st);
            else if (layout == k256) launch_layout<8, 1, true, false>(g, t, st);
            else launch_layout<4, 2, true, false>(g, t, st);
        }
        WK_LAUNCH_CHECK();
        if (!plan.merge) return WK_OK;
    } else {
        // more frames than the table holds: the same ranges as separate launches
        AttnArgs b = a;   // the rows behind the chunk, every query
        b.K += (size_t)start * row_bytes;
        b.V += (size_t)start * row_bytes;
        b.N_kv = N_kv - start;
        b.kv_start = start;
        b.part_slot = 1;
        wk_status rc = launch_plain(b, dtype, st);
        if (rc != WK_OK) return rc;
        for (int f = 0; f < frames; ++f) {   // rows up to the end of frame f of the chunk, that frame's queries
            AttnArgs p = a;
            p.N_q = frame_T;
            p.q_off = f * frame_T;
            p.N_kv = denoise_row0 + (f + 1) * frame_T;
            p.part_slot = 0;
            rc = launch_plain(p, dtype, st);
            if (rc != WK_OK) return rc;
        }
    }
    AttnArgs m = a;
    m.splits = 2;
    const size_t rows = (size_t)H * N_q;
    if (dtype == WK_F32)
        hipLaunchKernelGGL(k_attn_merge<WK_F32>, dim3((unsigned)((rows + 15) / 16)), dim3(256), 0, st, m);
    else
        hipLaunchKernelGGL(k_attn_merge<WK_BF16>, dim3((unsigned)((rows + 15) / 16)), dim3(256), 0, st, m);
    WK_LAUNCH_CHECK();
    return WK_OK;
}

extern "C" wk_status wk_chunk_lse(const wk_store_desc *store, const void *Q, int32_t N_q, float scale,
                                  float *lse_out, void *hip_stream) {
    if (!store || !Q || !lse_out) return WK_ERR_INVALID_ARG;
    if (store->M < 0 || store->H < 1 || N_q < 0 || store->max_tok < 0) return WK_ERR_INVALID_ARG;
    if (store->dtype != WK_F32 && store->dtype != WK_BF16) return WK_ERR_INVALID_ARG;
    if (!(scale >= 0.f) || std::isinf(scale)) return WK_ERR_INVALID_ARG;
    if (store->d != WK_D) return WK_ERR_UNSUPPORTED;
    if (store->dtype == WK_BF16 && store->max_tok > kMaxRowsBf16) return WK_ERR_UNSUPPORTED;   // 32-bit byte offsets
    if (store->M == 0 || N_q == 0) return WK_OK;
    if (!store->K_ptr || !store->n_tok) return WK_ERR_INVALID_ARG;
    AttnArgs a;
    a.Q = reinterpret_cast<const char *>(Q);
    a.K = a.V = nullptr;
    a.O = nullptr;
    a.lse = lse_out;
    a.H = store->H; a.N_q = N_q; a.N_kv = 0; a.kv_row_stride = 0;
    const float sc = scale == 0.f ? 1.f / std::sqrt((float)WK_D) : scale;
    a.scale_log2 = sc * 1.4426950408889634f;
    a.n_kv_dev = nullptr;
    a.splits = 1;
    a.part_o = nullptr;
    a.part_ml = nullptr;
    a.k_table = store->K_ptr;
    a.n_tok = store->n_tok;
    a.n_chunks = store->M;
    a.q_rows = N_q; a.q_off = 0; a.kv_start = 0; a.part_slot = -1;
    a.v_table = nullptr; a.ids = nullptr; a.n_ids = nullptr; a.R_max = 0; a.store_M = 0; a.max_tok = store->max_tok;
    hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
    const int q_per_wg = (store->dtype == WK_F32 ? kF32Waves : 8) * 32;
    const long long items = (long long)store->M * store->H * ((N_q + q_per_wg - 1) / q_per_wg);
    if (items + kXcds > 0x7fffffffLL) return WK_ERR_UNSUPPORTED;
    if (store->dtype == WK_F32) {
        return launch_f32(a, plan_f32((long long)store->H * store->M, N_q, (store->max_tok + kF32Keys - 1) / kF32Keys, 0).kg, st);
    }
    return launch_bf16(a, LaunchPlan{k256, 1}, nullptr, st);
}

extern "C" wk_status wk_attention_in_place(const void *Q, const void *K_native, const void *V_native,
                                           int32_t n_native, int32_t native_row_stride,
                                           const wk_store_desc *store, const int32_t *ids, const int32_t *n_ids,
                                           int32_t R_max, void *O, float *lse, int32_t N_q, float scale,
                                           void *hip_stream) {
    if (!store || !Q || !O) return WK_ERR_INVALID_ARG;
    if (store->M < 0 || store->H < 1 || store->max_tok < 0 || N_q < 0 || R_max < 0 || n_native < 0)
        return WK_ERR_INVALID_ARG;
    if (store->dtype != WK_F32 && store->dtype != WK_BF16) return WK_ERR_INVALID_ARG;
    if (!(scale >= 0.f) || std::isinf(scale)) return WK_ERR_INVALID_ARG;
    if (n_native > 0 && (!K_native || !V_native)) return WK_ERR_INVALID_ARG;
    if (R_max > 0 && store->M > 0 && (!ids || !store->K_ptr || !store->V_ptr || !store->n_tok))
        return WK_ERR_INVALID_ARG;
    if (store->d != WK_D || store->dtype != WK_BF16) return WK_ERR_UNSUPPORTED;
    if (R_max > kMaxSegments - 1) return WK_ERR_UNSUPPORTED;
    if (n_native >= (1 << 23) || store->max_tok >= (1 << 23)) return WK_ERR_UNSUPPORTED;   // 32-bit byte offsets
    if (n_native > native_row_stride) return WK_ERR_SHAPE;
    if (N_q == 0) return WK_OK;
    if ((long long)store->H * ((N_q + 255) / 256) + kXcds > 0x7fffffffLL) return WK_ERR_UNSUPPORTED;
    AttnArgs a;
    a.Q = reinterpret_cast<const char *>(Q);
    a.K = reinterpret_cast<const char *>(K_native);
    a.V = reinterpret_cast<const char *>(V_native);
    a.O = reinterpret_cast<char *>(O);
    a.lse = lse;
    a.H = store->H; a.N_q = N_q; a.N_kv = n_native; a.kv_row_stride = native_row_stride;
    const float sc = scale == 0.f ? 1.f / std::sqrt((float)WK_D) : scale;
    a.scale_log2 = sc * 1.4426950408889634f;
    a.n_kv_dev = nullptr;
    a.splits = 1;
    a.part_o = nullptr;
    a.part_ml = nullptr;
    a.k_table = store->K_ptr;
    a.n_tok = store->n_tok;
    a.n_chunks = 0;
    a.q_rows = N_q; a.q_off = 0; a.kv_start = 0; a.part_slot = -1;
    a.v_table = store->V_ptr; a.ids = ids; a.n_ids = n_ids; a.R_max = store->M > 0 ? R_max : 0; a.store_M = store->M;
    a.max_tok = store->max_tok;
    // 256- or 128-query workgroups, by the rule of wk_attention for the longest window the ids can give
    const long long longest = (long long)n_native + (long long)a.R_max * store->max_tok;
    const LaunchPlan plan = plan_bf16(a.H, N_q, (int)(longest < 64 ? 64 : (longest > 0x7fffffff ? 0x7fffffff : longest)), 0);
    const int q_per_wg = queries_per_wg(plan.layout);
    a.n_qtiles = (N_q + q_per_wg - 1) / q_per_wg;
    if (!wk::fits_launch((long long)a.H * a.n_qtiles + kXcds, kModel[plan.layout].qw * kModel[plan.layout].kg * 64)) return WK_ERR_UNSUPPORTED;
    a.per_xcd = (a.H * a.n_qtiles + kXcds - 1) / kXcds;
    const wk_status rc = allow_large_lds();
    if (rc != WK_OK) return rc;
    hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
    const bool trips = trips_in_place(n_native, a.R_max, store->max_tok);
    if (plan.layout == k256) trips ? launch_layout<8, 1, false, true, false, true>(a, SubTable{}, st) : launch_layout<8, 1, false, true>(a, SubTable{}, st);
    else if (plan.layout == k128Pair)
        trips ? launch_layout<4, 2, false, true, false, true>(a, SubTable{}, st) : launch_layout<4, 2, false, true>(a, SubTable{}, st);
    else launch_layout<4, 1, false, true>(a, SubTable{}, st);
    WK_LAUNCH_CHECK();
    return WK_OK;
}

extern "C" size_t wk_attention_workspace_bytes(int32_t H, int32_t N_q, int32_t N_kv, int32_t dtype) {
    if (H < 1 || N_q < 1 || N_kv < 1 || (dtype != WK_BF16 && dtype != WK_F32)) return 0;
    if ((long long)H * ((N_q + 31) / 32) > 0x7fffffffLL / kMaxSplits) return 0;
    if (dtype == WK_F32) {
        const int s = plan_f32(H, N_q, (N_kv + kF32Keys - 1) / kF32Keys, SIZE_MAX).splits;
        return s > 1 ? split_workspace_bytes(H, N_q, s) : 0;
    }
    const LaunchPlan plan = plan_bf16(H, N_q, N_kv, SIZE_MAX);
    return plan.splits > 1 ? split_workspace_bytes(H, N_q, plan.splits) : 0;
}

extern "C" int32_t wk_internal_attention_plan(int32_t H, int32_t N_q, int32_t N_kv, size_t workspace_bytes) {
    const LaunchPlan plan = plan_bf16(H, N_q, N_kv, workspace_bytes);
    return (int32_t)plan.layout * 100 + plan.splits;
}

extern "C" int32_t wk_internal_in_place_trips(int32_t n_native, int32_t R_max, int32_t max_tok) { return trips_in_place(n_native, R_max, max_tok) ? 1 : 0; }

extern "C" int32_t wk_internal_frame_mask_plan(int32_t H, int32_t N_q, int32_t N_kv, int32_t denoise_row0, int32_t frame_T) {
    if (N_q / frame_T + 1 > kMaxSub) return -1;
    const FramePlan p = plan_frames(H, N_q, N_kv, denoise_row0, frame_T);
    return (int32_t)p.layout + (p.merge ? 100 : 0);
}

extern "C" uint64_t wk_internal_interface() { return WK_INTERFACE; }   // of the wk.h this was compiled with

extern "C" const char *wk_status_string(wk_status s) {
    switch (s) {
    case WK_OK: return "ok";
    case WK_ERR_INVALID_ARG: return "invalid argument";
    case WK_ERR_SHAPE: return "inconsistent shape";
    case WK_ERR_RATIO: return "keep ratio out of range";
    case WK_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case WK_ERR_UNSUPPORTED: return "unsupported configuration";
    case WK_ERR_HIP: return "HIP runtime error";
    }
    return "unknown status";
}
