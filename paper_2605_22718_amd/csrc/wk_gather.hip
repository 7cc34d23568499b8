// Window assembly (paper Sec. 1: stored caches are reused as they are, not re-encoded; Sec. 4.2): the retrieved chunks' stored
// K/V rows are placed behind the native sliding-window rows, byte for byte.
//
// In the head-major layout every (head, chunk) pair is one contiguous byte range, so the gather
// is a set of H x (1 + R) straight copies.  One launch covers K and V.  A work unit is 8 to 32 KB of
// one head's K or V window; a workgroup walks units blockIdx.x, blockIdx.x + gridDim.x, ...: with
// the default grid that is one unit each, with a capped grid (a prefetch that runs beside other
// kernels and is bound by the host link anyway) a few workgroups stream the whole window.  The
// source of each 16-byte vector is found from the retrieved chunks' prefix offsets, built per wave in its lanes (per workgroup in LDS
// for more than 63 chunks) from the device-resident ids (which never visit the host); the waves of
// eight workgroups a compute unit, a request each, cover the latency of HBM and of reads from a pinned-host store over the host link.  Loads and stores are nontemporal (the data is touched once here), rows
// are 16 or 32 vectors so all index arithmetic is shifts on 32-bit values, and a unit that lies in
// one segment -- the usual case -- looks its segment up once: together with units of the right size these bring the kernel from
// 3.2 TB/s to 5.9 TB/s read + written (8 chunks of 40 heads x 2,340 tokens; the best plain device copy 6.4).  Small gathers are bound by
// the chain of look-ups before the first copy: units cover the retrieved rows only when the native ones are in place, unit
// numbers are 32-bit (4 chunks of 12 heads x 1,320 tokens: 20 -> 15 us), segments are in lanes (11.9 -> 11.3; 2 of 4 heads x 440, fp32, 5.2 -> 3.7, in smaller units 3.2).
#include <type_traits>

#include "wk_internal.h"

namespace {

constexpr int kMaxR = 1024;

// Work units: 256 threads with six vectors each where the copy is short, 512 with three beyond kLargeCopy bytes, the launch in order then
// sweeping the window closer to in sequence.  32 KB as 256 x 8, 24 KB as 256 x 6 and as 512 x 3: 8 chunks of 40 heads x 2,340 tokens (383 MB)
// 144, 142 and 130 us, 16 of 12 x 1,320 (130 MB) 54.9, 50.6 and 49.8, 3 of 40 x 700 (43 MB) 17.2, 14.7 and 18.7, 4 of 12 x 1,320 13.1, 13.0
// and 15.7 (512 x 2: 136, 51.4, 19.4, 15.4; 256 x 4: 133, 51.1, 19.3, 17.1; 256 x 1: 169, 66, 22, 17).  Between them either may be ahead: 256 x 6 and
// 512 x 3 take 27.1 and 25.5 us for 8 of 12 x 1,320 (65 MB), 32.2 and 32.2 for 10 (81 MB), 35.3 and 36.5 for 12 (97 MB), 41.5 and 38.0 for 5 of 40 x 1,040 (107 MB);
// above, 512 x 3 is: 50.3 and 47.4 for 7 of 16 x 2,340 (134 MB), 69.7 and 64.8 for 4 of 40 x 2,340 (192 MB).  A capped grid has 256 x 8.  Heads of less than a unit leave most of 512 threads idle (one row of 2^22 heads 17.6 ms, in
// 256 threads 9.9).
constexpr long long kLargeCopy = 128'000'000;
// Capped grids of fewer workgroups than this have all of a thread's loads under way, others one behind the other: 4 chunks of 40 heads x 2,340 rows from pinned memory with 8 workgroups
// 24.7 -> 56.6 GB/s, with 16 48.0 -> 56.7, but with 24 56.2 -> 54.9, with 256 57.2 -> 55.3 (4 of 12 x 1,320 55.8 -> 51.8); 32 and more reach 57 one behind the other.
constexpr long long kFewWorkgroups = 24;
// Copies of few units of 256 x 6 are made as 256 x 4 or 256 x 2: four or two latencies behind one another instead of six.  The bounds lie where pinned memory, which
// prefers few requests at a time, would lose more than a hundredth or two by it.  256 x 6, x 4 and x 2, from HBM in a graph / past the caches / from pinned memory: 16 units
// (4 heads x 100 rows) 3.2, 2.9, 2.6 / - / 10.9, 8.8, 7.6 us; 24 (4 x 280) 3.3, 3.0, 2.7 / 5.1, 4.1, 3.1 (4 x 200) / 14.4, 14.2, 14.6; 40 (4 x 440) 3.3, 3.0, 2.7 / 5.2, 4.2, 3.2 / 20.0, 19.9, 20.5;
// 152 (2 chunks of 4 x 440, fp32) 3.7, 3.4, 3.2 / 5.8, 4.9, 4.1 / 67.7, 68.8, 70.6; 336 (12 x 1,320) 6.8, 5.7, 5.1 / 7.4, 5.5, - / 148.6, 149.9, 178.6; 352 (16 x 1,000) 6.9, 5.8, - / - /
// 150.2, 151.7, -; but 456 (2 of 12 x 880) 8.0, 6.7, - / 7.9, 6.9, - / 196.8, 202.0, -, 672 (2 of 12 x 1,320) 9.4, 7.8, - / 9.4, 8.3, - / 296.7, 336.6, -.
// In 256 x 4 the first load tells where the store is, and from HBM the other three come together, two latencies as in 256 x 2: 40 units warm / past the caches / pinned 3.5, 4.2, 19.4 -> 3.4, 3.5, 19.6
// (256 x 2: 2.9, 3.2, 20.0), 152 5.0, 5.0, 68.3 -> 4.4, 4.2, 68.3 (4.2, 4.1, 70.0), 144 (12 x 500) 4.7, 4.8, 58.9 -> 4.2, 3.8, 58.9 (4.0, 4.0, 60.6), 336 6.2, 5.7, 149.1 -> 5.3, 5.5, 149.3.
constexpr long long kFewUnits = 360, kFewestUnits = 24;

typedef unsigned int uvec4 __attribute__((ext_vector_type(4)));   // a 16-byte vector the nontemporal builtins accept
typedef const __attribute__((address_space(1))) uvec4 *gvec4;     // in global memory, which a pointer put together from its halves does not tell

struct GatherArgs {
    const void *const *K_ptr;
    const void *const *V_ptr;
    const int32_t *n_tok;
    int M, max_tok, H;
    const int32_t *ids;
    const int32_t *n_ids;
    int R_max;
    const char *K_native;
    const char *V_native;
    int n_native;
    char *K_win;
    char *V_win;
    int win_capacity;
    int32_t *n_win;
    int vec_per_row;  // 16 (bf16) or 32 (fp32)
    int first_row;       // where the copy begins: 0, or behind native rows that are in place already
    int units_per_head;  // work units covering win_capacity-bounded rows of one head from there
};

__device__ inline void wait() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // for all loads and stores

constexpr int kLaneSegments = 64;   // native rows and up to 63 chunks: a lane each

// A segment of the window: 0 = native rows (null: already in place), 1.. = retrieved chunks in the order of ids.
struct Segment { const char *k, *v; int len; };

__device__ inline Segment segment_at(const GatherArgs &a, int s) {   // s < 1 + the count of ids: those behind it are never read
    if (s == 0) return Segment{a.K_native, a.V_native, a.n_native};
    Segment e{nullptr, nullptr, 0};
    const int id = a.ids[s - 1];
    if (id >= 0 && id < a.M) {
        const int len = a.n_tok[id];
        // a chunk that claims more rows than the descriptor's bound is skipped, like an id outside the
        // store: its length is the stride between its heads, so it cannot be cut short, and the window
        // was sized by the host for max_tok rows per chunk
        e.k = reinterpret_cast<const char *>(a.K_ptr[id]);
        e.v = reinterpret_cast<const char *>(a.V_ptr[id]);
        e.len = len < 0 || len > a.max_tok ? 0 : len;
    }
    return e;
}

// The look-ups.  IN_LANES (up to kLaneSegments): every wave has the segments in its lanes, places them by prefix sums in the vector pipe and
// finds a row's by counting the lanes that end before it: no LDS, no barrier, no search, which took 1.3 us of a small gather's 8.  Otherwise dynamic
// LDS holds, per segment, the base address of its K block and V block, its length and the first window row after it.
// U: the type of unit numbers, 32 bits except for a capped grid over 2^31 units or more (heads without end and next to no
// rows; the windows of anything else would not fit the device).  A 64-bit division takes longer than a unit's look-ups.
// PACED: a thread's stores wait for one another, as its loads do but where TOGETHER.
template <typename U, int THREADS, int VECS, bool IN_LANES, bool PACED, bool TOGETHER = false>
__global__ __launch_bounds__(THREADS, VECS > 6 ? 6 : 8) void k_gather(GatherArgs a) {
    constexpr unsigned kUnit = THREADS * VECS;   // 16-byte vectors
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int cap = a.R_max + 1;
    const char **seg_k = reinterpret_cast<const char **>(lds);
    const char **seg_v = seg_k + cap;
    int *seg_end = reinterpret_cast<int *>(seg_v + cap);
    int *seg_len = seg_end + cap;
    const int tid = threadIdx.x, lane = tid & 63;
    const size_t row_bytes = (size_t)a.vec_per_row * 16;

    int n = a.n_ids ? *a.n_ids : a.R_max;
    n = n < 0 ? 0 : (n > a.R_max ? a.R_max : n);
    const int nseg = n + 1;
    Segment mine{nullptr, nullptr, 0};
    int my_end = 0, total_rows;
    if constexpr (IN_LANES) {
        if (lane < nseg) mine = segment_at(a, lane);
        my_end = wk::wave_prefix(mine.len);
        total_rows = __builtin_amdgcn_readlane(my_end, 63);
    } else {
        for (int t = tid; t < nseg; t += THREADS) {
            const Segment e = segment_at(a, t);
            seg_len[t] = e.len;
            seg_k[t] = e.k;
            seg_v[t] = e.v;
        }
        __syncthreads();
        if (tid == 0) {
            int acc = 0;
            for (int t = 0; t < nseg; ++t) {
                acc += seg_len[t];
                seg_end[t] = acc;
            }
        }
        __syncthreads();
        total_rows = seg_end[nseg - 1];
    }
    if (a.n_win && blockIdx.x == 0 && tid == 0) *a.n_win = total_rows;
    if (total_rows > a.win_capacity) total_rows = a.win_capacity;  // cannot happen after the host check
    // rows are 16 or 32 vectors: shifts, and 32-bit indices inside a head (capacity * 32 < 2^31 is
    // checked on the host)
    const int row_shift = a.vec_per_row == 16 ? 4 : 5;
    const unsigned total_vec = (unsigned)total_rows << row_shift, first_vec = (unsigned)a.first_row << row_shift;
    const U units = (U)a.units_per_head * (U)a.H * 2u;
    // smallest s in [lo, hi] with row < its end
    auto segment_of = [&](int row, int lo, int hi) {
        if constexpr (IN_LANES) return (int)__popcll(__ballot(my_end <= row));   // (a row that all lanes ask for, of a segment)
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (row < seg_end[mid]) hi = mid; else lo = mid + 1;
        }
        return lo;
    };
    struct Source { const char *base; int begin, len; };   // of a segment
    auto source_of = [&](int sg, bool is_v) {
        if constexpr (IN_LANES) {
            const int len = __builtin_amdgcn_readlane(mine.len, sg);
            const uint64_t at = reinterpret_cast<uint64_t>(is_v ? mine.v : mine.k);
            const uint64_t base = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(at >> 32), sg) << 32 | (uint32_t)__builtin_amdgcn_readlane((int)at, sg);
            return Source{reinterpret_cast<const char *>(base), __builtin_amdgcn_readlane(my_end, sg) - len, len};
        } else {
            return Source{(is_v ? seg_v : seg_k)[sg], sg == 0 ? 0 : seg_end[sg - 1], seg_len[sg]};
        }
    };

    for (U u = blockIdx.x; u < units; u += gridDim.x) {
        const unsigned hz = (unsigned)(u / (U)a.units_per_head), unit = (unsigned)(u - (U)hz * (U)a.units_per_head);
        const unsigned v0 = first_vec + unit * kUnit;
        if (v0 >= total_vec) continue;
        const int h = (int)(hz % (unsigned)a.H);
        const bool is_v = hz >= (unsigned)a.H;
        uvec4 *win = reinterpret_cast<uvec4 *>((is_v ? a.V_win : a.K_win) + (size_t)h * a.win_capacity * row_bytes);
        // the unit's rows usually lie in one segment: look that up once
        const unsigned v_last = min(v0 + kUnit, total_vec) - 1;
        const int s_first = segment_of((int)(v0 >> row_shift), 0, nseg - 1);
        const int s_last = segment_of((int)(v_last >> row_shift), s_first, nseg - 1);
        // where the unit's vectors come from; null: nowhere
        gvec4 at[VECS];
        auto from = [&](const Source &src) {   // of the unit's first vector, were it in the segment
            return (gvec4)(reinterpret_cast<const uvec4 *>(src.base) + ((((ptrdiff_t)h * src.len - src.begin) << row_shift) + v0));
        };
#pragma unroll
        for (int i = 0; i < VECS; ++i) at[i] = nullptr;
        if constexpr (IN_LANES) {
            for (int sg = s_first; sg <= s_last; ++sg) {   // seldom more than one
                const Source src = source_of(sg, is_v);
                if (!src.base) continue;
                const gvec4 rows = from(src);
                const int first = (src.begin << row_shift) - (int)v0, end = min((src.begin + src.len) << row_shift, (int)total_vec) - (int)v0;   // in the unit
#pragma unroll
                for (int i = 0; i < VECS; ++i) {
                    const int v = tid + i * THREADS;
                    if (v >= first && v < end) at[i] = rows + v;
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < VECS; ++i) {
                const unsigned v = v0 + tid + i * THREADS;
                if (v >= total_vec) continue;
                const Source src = source_of(s_first == s_last ? s_first : segment_of((int)(v >> row_shift), s_first, s_last), is_v);
                if (src.base) at[i] = from(src) + (v - v0);
            }
        }
        uvec4 buf[VECS];
        bool near = TOGETHER;   // VECS == 4: the store is in HBM, as the first load tells
        const long long asked = VECS == 4 ? clock64() : 0;
#pragma unroll
        for (int i = 0; i < VECS; ++i) {   // one after the other, see the plan
            if (!near) wait();
            if (at[i]) buf[i] = __builtin_nontemporal_load(at[i]);   // (streamed once: kept out of the caches' way)
            if (VECS == 4 && i == 0) {
                wait();
                near = __builtin_amdgcn_readfirstlane((int)(clock64() - asked < wk::kNearCycles));
            }
        }
        if constexpr (!PACED) wait();   // (once: behind a branch the compiler waits for everything in front of each store)
#pragma unroll
        for (int i = 0; i < VECS; ++i) {
            if constexpr (PACED) wait();
            if (at[i]) __builtin_nontemporal_store(buf[i], win + v0 + tid + i * THREADS);
        }
    }
}

// One workgroup per unit, as far as a cap on workgroups and a launch's 2^32 threads allow: behind them workgroups take further units.
//
// A thread's loads wait for one another, but in grids of few units or workgroups (above): asked for together, rows come a little sooner from HBM but later from host memory, and where a store lies only the device
// knows (in units of 256 x 6, where a first load that tells does not pay: 2 chunks of 4 heads x 440 rows, fp32, 3.77 us one by one and 3.44 together, 8 of 40 x 2,340 122.3 and 124.6; one of 12 x 1,320 in pinned memory 148 and
// 183, two 301 and 339).  Its stores wait where the whole copy is under way at once but more than a workgroup a compute unit: 4 chunks of 12 heads x 1,320 rows 12.7 us
// without, 11.3 with it, 3 of 40 x 700 16.1 and 14.9, 4 of 24 x 760 14.0 and 12.8; less or more than that they don't: 3.77 and 4.28, 8 of 12 x 1,320 23.9 and 25.9,
// 8 of 40 x 2,340 122.3 and 125.5.  (With look-ups in LDS and both waiting at all sizes: 5.27, 12.1, 15.5, 13.3, 27.4 and 127.7.)
struct GatherPlan {
    int threads, vecs;
    long long units_per_head, units, grid;
    bool paced() const { return vecs == 6 && units >= 256 && units <= 2048; }   // (256 threads with up to 64 registers: eight workgroups a compute unit)
};

GatherPlan plan_gather(long long cap_vec, long long H, int max_workgroups) {   // cap_vec: 16-byte vectors to copy of a head's K, at most
    GatherPlan p{256, 6, 0, 0, 0};
    if (max_workgroups > 0) p.vecs = 8;
    else if (cap_vec >= 512 * 3 && (double)cap_vec * (double)H * 32 > (double)kLargeCopy) p = GatherPlan{512, 3, 0, 0, 0};
    const long long units = (cap_vec + 256 * 6 - 1) / (256 * 6) * H * 2;
    if (p.vecs == 6 && units <= kFewUnits) p.vecs = units <= kFewestUnits ? 2 : 4;
    const long long unit = p.threads * p.vecs;
    p.units_per_head = cap_vec > 0 ? (cap_vec + unit - 1) / unit : 1;   // nothing to copy: one workgroup still reports the (zero) length
    p.units = p.units_per_head * H * 2;
    p.grid = max_workgroups > 0 && p.units > max_workgroups ? max_workgroups : p.units;
    if (!wk::fits_launch(p.grid, p.threads)) p.grid = UINT32_MAX / p.threads;
    return p;
}

}  // namespace

extern "C" int64_t wk_internal_gather_threads(int32_t H, int64_t rows, int32_t dtype, int32_t max_workgroups) {
    const GatherPlan p = plan_gather(rows * (int64_t)(WK_D * wk::esize(dtype) / 16), H, max_workgroups);
    return p.grid * p.threads;
}

wk_status wk::gather_launch(const wk_store_desc *store, const int32_t *ids, const int32_t *n_ids, int32_t R_max,
                            const void *K_native, const void *V_native, int32_t n_native, void *K_win,
                            void *V_win, int32_t win_capacity, int32_t *n_win, int32_t max_workgroups,
                            hipStream_t stream) {
    if (!store || !K_win || !V_win) return WK_ERR_INVALID_ARG;
    if (R_max < 0 || n_native < 0 || win_capacity < 0 || store->M < 0 || store->max_tok < 0 || store->H < 1)
        return WK_ERR_INVALID_ARG;
    if (max_workgroups < 0) return WK_ERR_INVALID_ARG;
    if (store->dtype != WK_F32 && store->dtype != WK_BF16) return WK_ERR_INVALID_ARG;
    if (R_max > 0 && (!ids || !store->K_ptr || !store->V_ptr || !store->n_tok)) return WK_ERR_INVALID_ARG;
    if ((K_native == nullptr) != (V_native == nullptr)) return WK_ERR_INVALID_ARG;
    if (store->d != WK_D || R_max > kMaxR) return WK_ERR_UNSUPPORTED;
    if ((int64_t)n_native + (int64_t)R_max * store->max_tok > (int64_t)win_capacity) return WK_ERR_SHAPE;
    if ((int64_t)win_capacity * 32 > 0x7fffffffLL) return WK_ERR_UNSUPPORTED;   // 32-bit vector indices inside a head
    GatherArgs a;
    a.K_ptr = store->K_ptr; a.V_ptr = store->V_ptr; a.n_tok = store->n_tok;
    a.M = store->M; a.max_tok = store->max_tok; a.H = store->H;
    a.ids = ids; a.n_ids = n_ids; a.R_max = R_max;
    a.K_native = reinterpret_cast<const char *>(K_native);
    a.V_native = reinterpret_cast<const char *>(V_native);
    a.n_native = n_native;
    a.K_win = reinterpret_cast<char *>(K_win);
    a.V_win = reinterpret_cast<char *>(V_win);
    a.win_capacity = win_capacity;
    a.n_win = n_win;
    a.vec_per_row = (int)(WK_D * wk::esize(store->dtype) / 16);
    a.first_row = K_native ? 0 : n_native;
    const long long cap_vec = (long long)(n_native - a.first_row + (int64_t)R_max * store->max_tok) * a.vec_per_row;
    const size_t lds_bytes = R_max < kLaneSegments ? 0 : (size_t)(R_max + 1) * (2 * sizeof(char *) + 2 * sizeof(int));
    const GatherPlan p = plan_gather(cap_vec, store->H, max_workgroups);
    if (max_workgroups == 0 && p.units > 0x7fffffffLL) return WK_ERR_UNSUPPORTED;
    a.units_per_head = (int)p.units_per_head;
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3((unsigned)p.grid), dim3(p.threads), lds_bytes, stream, a); };
    // (32-bit unit numbers: one plus a grid stays below 2^32)
    auto launch_by = [&](auto in_lanes) {
        constexpr bool L = decltype(in_lanes)::value;
        if (max_workgroups > 0 && p.grid < kFewWorkgroups)
            p.units <= 0x7fffffffLL ? launch(k_gather<uint32_t, 256, 8, L, false, true>) : launch(k_gather<uint64_t, 256, 8, L, false, true>);
        else if (max_workgroups > 0) p.units <= 0x7fffffffLL ? launch(k_gather<uint32_t, 256, 8, L, false>) : launch(k_gather<uint64_t, 256, 8, L, false>);
        else if (p.threads == 512) launch(k_gather<uint32_t, 512, 3, L, false>);
        else if (p.vecs == 2) launch(k_gather<uint32_t, 256, 2, L, false>);
        else if (p.vecs == 4) launch(k_gather<uint32_t, 256, 4, L, false>);
        else if (p.paced()) launch(k_gather<uint32_t, 256, 6, L, true>);
        else launch(k_gather<uint32_t, 256, 6, L, false>);
    };
    R_max < kLaneSegments ? launch_by(std::true_type{}) : launch_by(std::false_type{});
    WK_LAUNCH_CHECK();
    return WK_OK;
}

extern "C" wk_status wk_gather_window(const wk_store_desc *store, const int32_t *ids, const int32_t *n_ids,
                                      int32_t R_max, const void *K_native, const void *V_native,
                                      int32_t n_native, void *K_win, void *V_win, int32_t win_capacity,
                                      int32_t *n_win, void *hip_stream) {
    return wk::gather_launch(store, ids, n_ids, R_max, K_native, V_native, n_native, K_win, V_win, win_capacity,
                             n_win, 0, reinterpret_cast<hipStream_t>(hip_stream));
}

namespace {

constexpr int kThreads = 256, kVecPerThread = 8, kVecPerBlock = kThreads * kVecPerThread;

// Straight copy with ordinary (cached) 16-byte loads and stores, one vector per lane and pass: the
// access pattern of the tile loads in the attention kernels, with a byte count known exactly.
__global__ __launch_bounds__(kThreads) void k_copy_plain(const uint4 *__restrict__ src, uint4 *__restrict__ dst,
                                                         long long n_vec) {
    const long long per_block = (long long)kThreads * kVecPerThread;
    for (long long base = (long long)blockIdx.x * per_block; base < n_vec; base += (long long)gridDim.x * per_block) {
        uint4 buf[kVecPerThread];
#pragma unroll
        for (int i = 0; i < kVecPerThread; ++i) {
            const long long v = base + threadIdx.x + (long long)i * kThreads;
            if (v < n_vec) buf[i] = src[v];
        }
#pragma unroll
        for (int i = 0; i < kVecPerThread; ++i) {
            const long long v = base + threadIdx.x + (long long)i * kThreads;
            if (v < n_vec) dst[v] = buf[i];
        }
    }
}

}  // namespace

extern "C" wk_status wk_calibration_copy(void *dst, const void *src, size_t bytes, void *hip_stream) {
    if (!dst || !src || bytes % 16 != 0) return WK_ERR_INVALID_ARG;
    if (reinterpret_cast<uintptr_t>(dst) % 16 != 0 || reinterpret_cast<uintptr_t>(src) % 16 != 0)
        return WK_ERR_INVALID_ARG;
    if (bytes == 0) return WK_OK;
    const long long n_vec = (long long)(bytes / 16);
    long long grid = (n_vec + kVecPerBlock - 1) / kVecPerBlock;
    if (grid > 0x7fffffffLL) grid = 0x7fffffffLL;
    hipLaunchKernelGGL(k_copy_plain, dim3((unsigned)grid), dim3(kThreads), 0,
                       reinterpret_cast<hipStream_t>(hip_stream), reinterpret_cast<const uint4 *>(src),
                       reinterpret_cast<uint4 *>(dst), n_vec);
    WK_LAUNCH_CHECK();
    return WK_OK;
}

extern "C" wk_status wk_host_device_pointer(void *host_ptr, void **device_ptr) {
    if (!host_ptr || !device_ptr) return WK_ERR_INVALID_ARG;
    void *dp = nullptr;
    if (hipHostGetDevicePointer(&dp, host_ptr, 0) != hipSuccess) {
        (void)hipGetLastError();
        return WK_ERR_HIP;
    }
    *device_ptr = dp;
    return WK_OK;
}
