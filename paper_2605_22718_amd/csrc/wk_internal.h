// Internal helpers shared by the HIP translation units of libwk (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "wk.h"

#define WK_D 128  // head dimension every kernel is written for

#define WK_LAUNCH_CHECK()                                   \
    do {                                                    \
        if (hipGetLastError() != hipSuccess) return WK_ERR_HIP; \
    } while (0)

// Not part of the interface: the tests pin with these that a shape takes the path it is there for.  How bf16 attention would
// be launched (0: 256 queries per workgroup, 1: 128 in pairs of tiles, 2: 128), under a frame mask (+ 100: as two key ranges, else as windows
// with a gap; -1: more frames than the table of launches holds); whether attention in place takes the hand-scheduled loop inside segments;
// head ranges of the similarity GEMM; threads that assemble a window of which
// `rows` a head are copied; launches of the compaction that writes `rows` a head.
extern "C" int32_t wk_internal_attention_plan(int32_t H, int32_t N_q, int32_t N_kv, size_t workspace_bytes);   // layout * 100 + key ranges
extern "C" int32_t wk_internal_frame_mask_plan(int32_t H, int32_t N_q, int32_t N_kv, int32_t denoise_row0, int32_t frame_T);
extern "C" int32_t wk_internal_in_place_trips(int32_t n_native, int32_t R_max, int32_t max_tok);
extern "C" int32_t wk_internal_gemm_head_ranges(const wk_compress_desc *desc);
extern "C" int32_t wk_internal_compact_launches(int64_t rows);
extern "C" int64_t wk_internal_gather_threads(int32_t H, int64_t rows, int32_t dtype, int32_t max_workgroups);

namespace wk {

__host__ __device__ inline size_t esize(int dtype) { return dtype == WK_BF16 ? 2 : 4; }

// A launch has fewer than 2^32 threads: the runtime drops the bits above without an error.
inline bool fits_launch(long long workgroups, int threads) { return workgroups * threads <= UINT32_MAX; }

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Once per device and process: true if `flags` did not yet have the current device's bit (the caller then
// does its per-device set-up, e.g. raising a kernel's dynamic-LDS limit, and calls it done with mark_device).
// A lost race only repeats an idempotent set-up.  Devices beyond 63 always report "not yet".
inline bool device_needs_setup(const std::atomic<uint64_t> &flags, int &dev) {
    if (hipGetDevice(&dev) != hipSuccess) dev = -1;
    return dev < 0 || dev > 63 || !((flags.load(std::memory_order_acquire) >> dev) & 1u);
}
inline void mark_device(std::atomic<uint64_t> &flags, int dev) {
    if (dev >= 0 && dev <= 63) flags.fetch_or(uint64_t(1) << dev, std::memory_order_release);
}

// wk_gather_window with a cap on the number of workgroups (0 = one per work unit)
wk_status gather_launch(const wk_store_desc *store, const int32_t *ids, const int32_t *n_ids, int32_t R_max,
                        const void *K_native, const void *V_native, int32_t n_native, void *K_win, void *V_win,
                        int32_t win_capacity, int32_t *n_win, int32_t max_workgroups, hipStream_t stream);

// a pointer that is the same in every lane, as a scalar
__device__ inline const char *uniform_ptr(const char *p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const char *>(((uint64_t)hi << 32) | lo);
}

// Inclusive prefix sums over the wave, in the vector pipe (shuffles go through the LDS): shifts inside rows of 16 lanes, then the rows' last
// lanes to the rows behind them.
__device__ inline int wave_prefix(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15, rows 1 and 3
    return x + __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31, rows 2 and 3
}

// A load that comes within so many cycles, about 1.5 us, came from HBM (0.3 to 1 us) and not from host memory (1.1 to 2.6, and then its turn on the link).
constexpr int kNearCycles = 3500;

// 16 lanes share one 128-element row; each lane owns elements 8*sub .. 8*sub+7.
constexpr int kRowLanes = 16;

template <int DT>
__device__ inline void load_row8(const void *row_base, int sub, float (&v)[8]) {
    if constexpr (DT == WK_BF16) {
        const uint4 u = reinterpret_cast<const uint4 *>(row_base)[sub];
        const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] = __uint_as_float(w[i] << 16);
            v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    } else {
        const float4 a = reinterpret_cast<const float4 *>(row_base)[2 * sub];
        const float4 b = reinterpret_cast<const float4 *>(row_base)[2 * sub + 1];
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    }
}

// sum over the 16 lanes of a row group (groups are aligned to 16 lanes)
__device__ inline double row_group_sum(double x) {
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

}  // namespace wk
