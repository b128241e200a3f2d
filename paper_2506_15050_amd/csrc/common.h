// Internal helpers shared by the HIP translation units of libtppo (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tppo.h"

#define TPPO_VERSION 100

namespace tppo {

constexpr int kWave = 64;

static inline bool is_aligned(const void* p, size_t a) {
    return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0;
}

static constexpr size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

static inline int launch_result() {
    return hipGetLastError() == hipSuccess ? TPPO_OK : TPPO_ERR_LAUNCH;
}

__device__ __forceinline__ void set_status(int32_t* status, int32_t bit) {
    if (status) atomicOr(status, bit);
}

// Loads of wave-uniform values through the scalar data cache (read-only data written before the launch).  Cheap
// when the line is there (kernel arguments, a header every wavefront reads); a MISS was measured at 4000-6000
// cycles with thousands of wavefronts in flight, several times a vector load's latency -- so per-tile data that
// a wavefront waits for goes through vector loads, and scalar loads are for what is fetched well ahead.
__device__ __forceinline__ int32_t load_uniform(const int32_t* p) {
    return *(const int32_t __attribute__((address_space(4)))*)(p);
}
__device__ __forceinline__ float load_uniform(const float* p) {
    return *(const float __attribute__((address_space(4)))*)(p);
}
__device__ __forceinline__ long long load_uniform(const long long* p) {
    return *(const long long __attribute__((address_space(4)))*)(p);
}

// Compute units of the current device (asked once per device; <= 0 when the runtime cannot say).
int device_compute_units();

// Sums and scans over a wavefront by data-parallel moves: row_shr 1, 2, 4, 8, then row_bcast 15 and 31, each a step of some cycles,
// where a shuffle is a trip through the LDS crossbar of more than a hundred.
// Data-parallel move: lane i receives x of the lane the control word names; lanes without a
// source (start of a row, a row that row_mask leaves out) receive 0.
constexpr int kRowShr1 = 0x111, kRowShr2 = 0x112, kRowShr4 = 0x114, kRowShr8 = 0x118;
constexpr int kWaveShr1 = 0x138, kRowBcast15 = 0x142, kRowBcast31 = 0x143;
template <int kCtrl, int kRowMask>
__device__ __forceinline__ int dpp_move(int x) {
    // where every row is written a lane without a source reads 0 by itself (bound_ctrl), and the destination
    // needs no initial value -- one instruction instead of two
    if constexpr (kRowMask == 0xF) return __builtin_amdgcn_mov_dpp(x, kCtrl, 0xF, 0xF, true);
    else return __builtin_amdgcn_update_dpp(0, x, kCtrl, kRowMask, 0xF, false);
}
template <int kCtrl, int kRowMask>
__device__ __forceinline__ float dpp_move(float x) {
    return __int_as_float(dpp_move<kCtrl, kRowMask>(__float_as_int(x)));
}
template <int kCtrl, int kRowMask>
__device__ __forceinline__ double dpp_move(double x) {
    return __hiloint2double(dpp_move<kCtrl, kRowMask>(__double2hiint(x)), dpp_move<kCtrl, kRowMask>(__double2loint(x)));
}
// sums over the lanes up to and including one's own: lane 63 has the wavefront's
template <class T>
__device__ __forceinline__ T wave_prefix(T x) {
    x += dpp_move<kRowShr1, 0xF>(x);
    x += dpp_move<kRowShr2, 0xF>(x);
    x += dpp_move<kRowShr4, 0xF>(x);
    x += dpp_move<kRowShr8, 0xF>(x);
    x += dpp_move<kRowBcast15, 0xA>(x);                              // lane 15 / 47 into rows 1 / 3
    x += dpp_move<kRowBcast31, 0xC>(x);                              // lane 31 into rows 2 and 3
    return x;
}

// the largest of non-negative numbers, the same in every lane
__device__ __forceinline__ int wave_max(int x) {
    x = max(x, dpp_move<kRowShr1, 0xF>(x));
    x = max(x, dpp_move<kRowShr2, 0xF>(x));
    x = max(x, dpp_move<kRowShr4, 0xF>(x));
    x = max(x, dpp_move<kRowShr8, 0xF>(x));
    x = max(x, dpp_move<kRowBcast15, 0xA>(x));
    x = max(x, dpp_move<kRowBcast31, 0xC>(x));
    return __builtin_amdgcn_readlane(x, kWave - 1);
}

// largest s in [lo, hi] with off[s] <= p  (off non-decreasing, off[lo] <= p)
__device__ __forceinline__ int find_segment(const int32_t* off, int lo, int hi, int p) {
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= p) lo = mid; else hi = mid - 1;
    }
    return lo;
}

}  // namespace tppo
