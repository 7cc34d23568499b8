// Window bookkeeping (paper Sec. 4.2: the sliding window has a sink, a retrieved, a recent and a
// denoising region; Sec. 5.1: 3 + 9 + 3 + 3 latent frames).
//
// Two parts.  wk_window_plan is host arithmetic: where the chunk being generated lives, which
// chunk leaves the ring and must go to the store first.  Physical layout per head, in rows:
//
//     [ sink chunks | ring of (recent_chunks + 1) chunk slots | R retrieved slots ]
//
// Attention is a sum over keys, so the order of regions inside the window is free; this order
// makes every valid prefix contiguous (ring slots fill in ascending order, and nothing is
// retrieved before the ring is full) and needs no copy when a denoised chunk becomes "recent":
// the roles rotate over the ring slots instead.
//
// wk_window_update refreshes the retrieved region in place on the device.  Consecutive steps of
// a smooth camera path want mostly the same chunks; only chunks that are not already resident
// are copied from the store (HBM or pinned host), into the slots of the chunks that left.  One
// small kernel turns (old slot table, wanted ids) into (new slot table, fetch list); a second
// copies the fetch list.
#include <type_traits>

#include "wk_internal.h"

namespace {

constexpr int kPlanThreads = 1024;
constexpr int kMaxSlots = 1024;
constexpr int kThreads = 256;
constexpr int kBlocksPerWg = 8;
constexpr int kBlocksInFlight = 256;   // 1 MB

// Workgroups for a list of `blocks` blocks: beyond 128 two blocks for each, beyond 512 more of them and one block in flight for
// each, at most kBlocksPerWg in turn.  (From pinned memory 300 blocks take 31.8 us with 128 workgroups, 35.3 with 256, and 1,320
// blocks 104.2 with 192, 105.3 with 256; 660 blocks from HBM 9.0, 8.6 and 8.4 us with 128, 192 and 256.)
__host__ __device__ inline long long fetch_grid(long long blocks) {
    const long long few = blocks < 128 ? blocks : (blocks <= 512 ? 128 : 192), many = (blocks + kBlocksPerWg - 1) / kBlocksPerWg;
    return few > many ? few : many;
}

typedef unsigned int uvec4 __attribute__((ext_vector_type(4)));   // a 16-byte vector the nontemporal builtins accept

struct PlanOut {   // head of the workspace
    int32_t n_fetch;
    int32_t n_used;
};

__global__ __launch_bounds__(kPlanThreads) void k_slot_plan(const int32_t *__restrict__ ids,
                                                            const int32_t *__restrict__ n_ids, int R, int M,
                                                            const int32_t *__restrict__ n_tok, int slot_tokens,
                                                            int32_t *__restrict__ slot_ids, int n_native,
                                                            int32_t *__restrict__ n_win, int32_t *__restrict__ n_fetched,
                                                            PlanOut *__restrict__ head, int32_t *__restrict__ fetch_slot,
                                                            int32_t *__restrict__ fetch_id) {
    __shared__ int raw[kMaxSlots], want[kMaxSlots], old[kMaxSlots], inc[kMaxSlots];
    __shared__ unsigned char ok[kMaxSlots], keep[kMaxSlots], res[kMaxSlots], fetch[kMaxSlots];
    __shared__ int s_n;
    const int s = threadIdx.x;   // one thread per slot / per wanted rank
    int n_in = n_ids ? *n_ids : R;
    n_in = n_in < 0 ? 0 : (n_in > R ? R : n_in);
    if (s < R) {
        old[s] = slot_ids[s];
        int id = s < n_in ? ids[s] : -1;
        if (id < 0 || id >= M || n_tok[id] != slot_tokens) id = -1;   // not placeable: dropped
        raw[s] = id;
    }
    if (s == 0) s_n = 0;
    __syncthreads();
    // drop repeats of an earlier rank; compact the rest in rank order
    if (s < R) {
        bool good = raw[s] >= 0;
        for (int t = 0; good && t < s; ++t) good = raw[t] != raw[s];
        ok[s] = good;
    }
    __syncthreads();
    if (s < R && ok[s]) {
        int pos = 0;
        for (int t = 0; t < s; ++t) pos += ok[t];
        want[pos] = raw[s];
        atomicAdd(&s_n, 1);
    }
    __syncthreads();
    const int n = s_n;
    // resident and wanted chunks keep their slot -- unless one sits at or beyond slot n
    // (a slot table that names one chunk twice keeps the first copy only)
    bool my_keep = false;
    if (s < R && old[s] >= 0) {
        for (int w = 0; w < n; ++w) my_keep |= want[w] == old[s];
        for (int t = 0; my_keep && t < s; ++t) my_keep = old[t] != old[s];
    }
    if (s < R) keep[s] = my_keep;
    const int rebuild = __syncthreads_or(my_keep && s >= n);
    if (s < n) {   // is the chunk of rank s already resident (in a kept slot)?
        bool r = false;
        for (int t = 0; t < R; ++t) r |= keep[t] && old[t] == want[s];
        res[s] = r;
    }
    __syncthreads();
    if (s < n && !res[s] && !rebuild) {   // newcomers in rank order
        int pos = 0;
        for (int w = 0; w < s; ++w) pos += !res[w];
        inc[pos] = want[s];
    }
    __syncthreads();
    int mine = -1;
    bool my_fetch = false;
    if (s < n) {
        if (rebuild) {
            mine = want[s];
            my_fetch = old[s] != mine;
        } else if (keep[s]) {
            mine = old[s];
        } else {
            int pos = 0;   // rank of this slot among the free ones below n
            for (int t = 0; t < s; ++t) pos += !keep[t];
            mine = inc[pos];
            my_fetch = true;
        }
    }
    if (s < R) {
        fetch[s] = my_fetch;
        slot_ids[s] = mine;
    }
    __syncthreads();
    if (my_fetch) {
        int pos = 0;
        for (int t = 0; t < s; ++t) pos += fetch[t];
        fetch_slot[pos] = s;
        fetch_id[pos] = mine;
    }
    if (s == 0) {
        int total = 0;
        for (int t = 0; t < n; ++t) total += fetch[t];
        head->n_fetch = total;
        head->n_used = n;
        if (n_win) *n_win = n_native + n * slot_tokens;
        if (n_fetched) *n_fetched = total;
    }
}

// Division by a number the host knows.  32 bits: with m = min(2^32 / d, 2^32 - 1), rounded down, n * m / 2^32 is the quotient
// or one less.  (In full they would take longer than a block's look-ups.)
struct Divider {
    uint64_t d;
    uint32_t m;
    __host__ explicit Divider(uint64_t by = 1) : d(by), m(by <= 1 ? 0xffffffffu : (uint32_t)((1ull << 32) / by)) {}
    __device__ uint32_t divide(uint32_t n, uint32_t &rest) const {
        uint32_t q = __umulhi(n, m);
        rest = n - q * (uint32_t)d;
        if (rest >= (uint32_t)d) {
            ++q;
            rest -= (uint32_t)d;
        }
        return q;
    }
    __device__ uint64_t divide(uint64_t n, uint64_t &rest) const {
        const uint64_t q = n / d;
        rest = n - q * d;
        return q;
    }
};

struct FetchArgs {
    const void *const *K_ptr;
    const void *const *V_ptr;
    const PlanOut *head;
    const int32_t *fetch_slot;
    const int32_t *fetch_id;
    char *K_win;
    char *V_win;
    int H, R, slot_tokens, n_native, win_capacity, vec_per_row;
    long long blocks;   // 4 KB blocks that cover one chunk's K, all heads (its V the same)
    Divider by_blocks, by_units, by_slot_vec;   // by that, by kBlocksPerWg blocks at a time, by the 16-byte vectors of one head
    bool wide, capped;
};

// The fetch list's chunks, K and V of each, are laid end to end in blocks of 4 KB (a chunk's heads are contiguous in the
// store), which the workgroups walk side by side.
//
// From HBM everything should be in flight at once; from pinned host memory, which bounds the call there, not: a
// burst for all of a chunk begins with a storm of address translations, and one chunk of 12 x 1,320 tokens takes
// 187 us with 32 KB in flight in each of 264 workgroups, 154 us (the copy engine: 151 us) with about 1 MB in flight in all.  So
// each workgroup times its first blocks: if they came within kNearCycles they came from HBM (a load takes 0.3 to 1 us there; 1.1
// to 2.6 us from the host, and then its turn on the link), and eight times as much is in flight from then on.  From HBM that
// chunk takes 11.2 us (10.3 us all at once, 12.6 us never more than 1 MB); two of 40 x 2,340 43 us either way.
// A grid that the caller caps (16 workgroups serve the host link) takes 32 KB per workgroup and trip.
//
// The threads of a block share its entry, head and first vector: scalar work; a thread only steps over the heads that
// begin inside the block.
using wk::kNearCycles;

template <typename I>
struct Fetch {
    const FetchArgs &a;
    I chunk_vec, slot_vec;   // 16-byte vectors of a chunk's K, of one head of it

    // D consecutive runs of kThreads vectors from vector `first` on; entry e = 2 * f + (0: K, 1: V)
    template <int D>
    __device__ __forceinline__ void load(uvec4 (&buf)[D], const char *src, I first) const {
#pragma unroll
        for (int i = 0; i < D; ++i) {   // past the end: the last vector again, and no store
            const I v = first + i * kThreads + threadIdx.x;
            buf[i] = __builtin_nontemporal_load(reinterpret_cast<const uvec4 *>(src) + (v < chunk_vec ? v : chunk_vec - 1));
        }
    }
    template <int D>
    __device__ __forceinline__ void store(const uvec4 (&buf)[D], int e, int row, I first) const {
        I in_head;
        const I h = a.by_slot_vec.divide(first, in_head);
        uvec4 *at = reinterpret_cast<uvec4 *>(e & 1 ? a.V_win : a.K_win) + ((size_t)h * a.win_capacity + row) * a.vec_per_row;
        if (in_head + D * kThreads <= slot_vec) {   // all in one head, the usual case
#pragma unroll
            for (int i = 0; i < D; ++i) __builtin_nontemporal_store(buf[i], at + in_head + i * kThreads + threadIdx.x);
            return;
        }
        in_head += threadIdx.x;
#pragma unroll
        for (int i = 0; i < D; ++i) {
            for (; in_head >= slot_vec; in_head -= slot_vec) at += (size_t)a.win_capacity * a.vec_per_row;
            if (first + i * kThreads + threadIdx.x < chunk_vec) __builtin_nontemporal_store(buf[i], at + in_head);
            in_head += kThreads;
        }
    }
    // a grid capped to fewer workgroups than that: units of kBlocksPerWg blocks of one entry, all in flight
    __device__ __forceinline__ void units(int n_fetch) const {
        const I total = 2 * (I)a.by_units.d * (I)n_fetch;
        for (I u = blockIdx.x; u < total; u += gridDim.x) {
            I unit;
            const int e = (int)a.by_units.divide(u, unit);
            const int id = a.fetch_id[e >> 1], row = a.n_native + a.fetch_slot[e >> 1] * a.slot_tokens;
            uvec4 buf[kBlocksPerWg];
            load(buf, reinterpret_cast<const char *>(e & 1 ? a.V_ptr[id] : a.K_ptr[id]), unit * (kBlocksPerWg * kThreads));
            store(buf, e, row, unit * (kBlocksPerWg * kThreads));
        }
    }
};

__global__ __launch_bounds__(kThreads) void k_slot_fetch(FetchArgs a) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int n_fetch = a.head->n_fetch;
    if (a.wide) {   // numbers beyond 32 bits
        const Fetch<uint64_t> fetch{a, (uint64_t)a.H * a.by_slot_vec.d, a.by_slot_vec.d};
        fetch.units(n_fetch);
        return;
    }
    const Fetch<uint32_t> fetch{a, (uint32_t)a.H * (uint32_t)a.by_slot_vec.d, (uint32_t)a.by_slot_vec.d};
    if (a.capped) {
        fetch.units(n_fetch);
        return;
    }
    // as many workgroups as the list needs, of those launched for R entries
    const uint32_t total = 2 * (uint32_t)a.by_blocks.d * (uint32_t)n_fetch, grid = (uint32_t)fetch_grid(total);
    if (blockIdx.x >= grid) return;
    const char **src_of = reinterpret_cast<const char **>(lds);   // [2 * n_fetch]: K and V of each entry
    int *row_of = reinterpret_cast<int *>(src_of + 2 * a.R);      // [n_fetch]: first window row of its slot
    for (int f = threadIdx.x; f < n_fetch; f += kThreads) {
        const int id = a.fetch_id[f];
        src_of[2 * f] = reinterpret_cast<const char *>(a.K_ptr[id]);
        src_of[2 * f + 1] = reinterpret_cast<const char *>(a.V_ptr[id]);
        row_of[f] = a.n_native + a.fetch_slot[f] * a.slot_tokens;
    }
    __syncthreads();
    // D blocks y, y + grid, ...: all requested before the first is stored
    long long landed = 0;
    auto blocks = [&](auto depth, uint32_t y, bool timed) __attribute__((always_inline)) {
        constexpr int D = decltype(depth)::value;
        uvec4 buf[D][1];
        uint32_t first[D];
        int e[D];
#pragma unroll
        for (int i = 0; i < D; ++i) {
            const uint32_t z = y + i * grid;
            uint32_t block;
            e[i] = (int)a.by_blocks.divide(z < total ? z : total - 1, block);
            first[i] = block * kThreads;
            fetch.load(buf[i], src_of[e[i]], first[i]);
            if (z >= total) first[i] = fetch.chunk_vec;
        }
        if (timed) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            landed = clock64();
        }
#pragma unroll
        for (int i = 0; i < D; ++i)
            if (first[i] < fetch.chunk_vec) fetch.store(buf[i], e[i], row_of[e[i] >> 1], first[i]);
    };
    uint32_t depth = kBlocksInFlight / grid, y = blockIdx.x;
    bool timed = true;
    const long long asked = clock64();
    while (y < total) {
        const uint32_t rounds = (total - y + grid - 1) / grid, d = depth < rounds ? depth : rounds;
        if (d > 4) {
            blocks(std::integral_constant<int, 8>{}, y, timed);
            y += 8 * grid;
        } else if (d > 2) {
            blocks(std::integral_constant<int, 4>{}, y, timed);
            y += 4 * grid;
        } else if (d > 1) {
            blocks(std::integral_constant<int, 2>{}, y, timed);
            y += 2 * grid;
        } else {
            blocks(std::integral_constant<int, 1>{}, y, timed);
            y += grid;
        }
        if (timed && landed - asked < kNearCycles) depth = 8 * kBlocksInFlight / grid;
        timed = false;
    }
}

}  // namespace

extern "C" wk_status wk_window_plan(const wk_window_desc *w, int64_t chunk_index, wk_window_step *out) {
    if (!w || !out || chunk_index < 0) return WK_ERR_INVALID_ARG;
    if (w->T < 1 || w->chunk_frames < 1 || w->sink_chunks < 0 || w->recent_chunks < 0 || w->R < 0 ||
        w->slot_tokens < 0)
        return WK_ERR_INVALID_ARG;
    const int64_t chunk_rows = (int64_t)w->chunk_frames * w->T;
    const int64_t ring_slots = (int64_t)w->recent_chunks + 1;
    const int64_t native_cap = ((int64_t)w->sink_chunks + ring_slots) * chunk_rows;
    const int64_t cap = native_cap + (int64_t)w->R * w->slot_tokens;
    if (cap > 0x7fffffffLL) return WK_ERR_UNSUPPORTED;
    out->denoise_rows = (int32_t)chunk_rows;
    out->retrieved_row0 = (int32_t)native_cap;
    out->win_capacity = (int32_t)cap;
    out->evict = 0;
    out->evict_row0 = 0;
    out->evict_chunk = -1;
    out->store_id = -1;
    if (chunk_index < w->sink_chunks) {   // one of the initial chunks: it is (part of) the sink
        out->denoise_row0 = (int32_t)(chunk_index * chunk_rows);
        out->n_native = (int32_t)((chunk_index + 1) * chunk_rows);
        out->M = 0;
        return WK_OK;
    }
    const int64_t k = chunk_index - w->sink_chunks;   // chunks that entered the ring before this one
    const int64_t slot = k % ring_slots;
    out->denoise_row0 = (int32_t)((w->sink_chunks + slot) * chunk_rows);
    const int64_t in_ring = k + 1 < ring_slots ? k + 1 : ring_slots;
    out->n_native = (int32_t)((w->sink_chunks + in_ring) * chunk_rows);
    if (k >= ring_slots) {   // the slot still holds chunk (chunk_index - ring_slots): store it first
        out->evict = 1;
        out->evict_row0 = out->denoise_row0;
        out->evict_chunk = chunk_index - ring_slots;
        const int64_t sid = k - ring_slots;
        if (sid > 0x7fffffffLL) return WK_ERR_UNSUPPORTED;
        out->store_id = (int32_t)sid;
    }
    const int64_t stored = k >= ring_slots ? k - ring_slots + 1 : 0;
    out->M = (int32_t)(stored > 0x7fffffffLL ? 0x7fffffffLL : stored);
    return WK_OK;
}

extern "C" size_t wk_window_update_workspace_bytes(int32_t R) {
    if (R < 0 || R > kMaxSlots) return 0;
    return 256 + wk::align_up((size_t)(R > 0 ? R : 1) * 2 * sizeof(int32_t), 256);
}

extern "C" wk_status wk_window_update(const wk_store_desc *store, const int32_t *ids, const int32_t *n_ids,
                                      int32_t R, int32_t slot_tokens, int32_t *slot_ids, int32_t n_native,
                                      void *K_win, void *V_win, int32_t win_capacity, int32_t *n_win,
                                      int32_t *n_fetched, void *workspace, size_t workspace_bytes,
                                      int32_t max_workgroups, void *hip_stream) {
    if (!store || !K_win || !V_win) return WK_ERR_INVALID_ARG;
    if (R < 0 || slot_tokens < 1 || n_native < 0 || win_capacity < 0 || max_workgroups < 0 || store->M < 0 ||
        store->H < 1)
        return WK_ERR_INVALID_ARG;
    if (store->dtype != WK_F32 && store->dtype != WK_BF16) return WK_ERR_INVALID_ARG;
    if (R > 0 && (!ids || !slot_ids)) return WK_ERR_INVALID_ARG;
    if (R > 0 && store->M > 0 && (!store->K_ptr || !store->V_ptr || !store->n_tok)) return WK_ERR_INVALID_ARG;
    if (store->d != WK_D || R > kMaxSlots) return WK_ERR_UNSUPPORTED;
    if ((int64_t)n_native + (int64_t)R * slot_tokens > (int64_t)win_capacity) return WK_ERR_SHAPE;
    if (slot_tokens > store->max_tok && store->M > 0) return WK_ERR_SHAPE;   // no chunk within the store's bound fits the slots
    const size_t need = wk_window_update_workspace_bytes(R);
    if (!workspace || workspace_bytes < need || reinterpret_cast<uintptr_t>(workspace) % 256 != 0)
        return WK_ERR_WORKSPACE;
    hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
    PlanOut *head = reinterpret_cast<PlanOut *>(workspace);
    int32_t *fetch_slot = reinterpret_cast<int32_t *>(reinterpret_cast<char *>(workspace) + 256);
    int32_t *fetch_id = fetch_slot + (R > 0 ? R : 1);
    hipLaunchKernelGGL(k_slot_plan, dim3(1), dim3(kPlanThreads), 0, st, ids, n_ids, (int)R, (int)store->M,
                       store->n_tok, (int)slot_tokens, slot_ids, (int)n_native, n_win, n_fetched, head, fetch_slot,
                       fetch_id);
    WK_LAUNCH_CHECK();
    if (R == 0 || store->M == 0) return WK_OK;
    FetchArgs a;
    a.K_ptr = store->K_ptr; a.V_ptr = store->V_ptr;
    a.head = head; a.fetch_slot = fetch_slot; a.fetch_id = fetch_id;
    a.K_win = reinterpret_cast<char *>(K_win);
    a.V_win = reinterpret_cast<char *>(V_win);
    a.H = store->H; a.R = R; a.slot_tokens = slot_tokens; a.n_native = n_native; a.win_capacity = win_capacity;
    a.vec_per_row = (int)(WK_D * wk::esize(store->dtype) / 16);
    const long long slot_vec = (long long)slot_tokens * a.vec_per_row;
    a.blocks = (a.H * slot_vec + kThreads - 1) / kThreads;
    a.by_blocks = Divider(a.blocks);
    a.by_units = Divider((a.blocks + kBlocksPerWg - 1) / kBlocksPerWg);
    a.by_slot_vec = Divider(slot_vec);
    // (block and unit numbers run past their ends by less than eight grids, vector numbers by less than eight blocks)
    a.wide = 2 * a.blocks * R > (1ll << 26) || a.blocks * kThreads > (1ll << 30);
    const long long units = 2 * (long long)a.by_units.d * R, wanted = a.wide ? units : fetch_grid(2 * a.blocks * R);
    a.capped = max_workgroups > 0 && wanted > max_workgroups;
    long long grid = a.capped ? max_workgroups : wanted;
    if (grid > 0x7fffffffLL) grid = 0x7fffffffLL;
    const size_t lds_bytes = (size_t)R * (2 * sizeof(char *) + sizeof(int));
    hipLaunchKernelGGL(k_slot_fetch, dim3((unsigned)grid), dim3(kThreads), lds_bytes, st, a);
    WK_LAUNCH_CHECK();
    return WK_OK;
}
