// tppo_value_head: V(s_t) = w . h_t + bias for a list of hidden rows -- the
// critic-side mirror of the LM head (the value model of Sec. 2.2 ends in a
// projection to one scalar), producing the v_new that Eq. (valueloss) consumes.
// A gathered matrix-vector product: every row is read once (2 H bytes, bf16), so the kernel is bound by HBM.  A
// wavefront takes kRows rows at once, lanes on consecutive 16 bytes of each; fp32 accumulation, wave reduction.
#include "common.h"

namespace tppo {

constexpr int kVhThreads = 256, kVhWaves = kVhThreads / kWave;
constexpr int kVhMaxH = 16384;
constexpr int64_t kVhMaxGroups = 1 << 20;         // (more rows than 16 million: several turns per wavefront)
constexpr int64_t kVhFewRows = 256 * 3 * 8;

typedef uint32_t vh_chunk __attribute__((ext_vector_type(4)));
typedef uint32_t vh_weights __attribute__((ext_vector_type(4), aligned(2)));   // w_value may start anywhere

// kRows rows per wavefront: one 16-byte load per row and step, two steps in flight, and the weights, which every
// wavefront of the CU reads and the vector cache holds, fetched once for all of them.  One group of rows per
// wavefront and no loop over groups: nothing waits for a workgroup's slowest row.
// Measured, hidden states that no cache holds: 94639 rows of H = 5120, 140 us = 6.9 TB/s; of H = 1024, 30 us = 6.4; 20000 of H = 3584,
// 24 us.  One row per wavefront, two plain loads in flight, the weights as fp32 in LDS and a persistent grid took
// 221, 52 and 40 us; plain instead of non-temporal loads cost 14 %, one row per wavefront 13 % at H = 1024.  A row's sum over the lanes by
// data-parallel moves instead of shuffles, rows in a cache: 4000 of H = 512 2.8 -> 2.6 us, 6000 of H = 2048 5.4 -> 5.1.  (One row a wavefront and
// four steps in flight: 2000 of H = 5120 6.1 -> 5.6, 4000 of them 7.7 -> 8.6, of H = 512 2.6 -> 3.2.)
template <int kRows>
__global__ __launch_bounds__(kVhThreads) void value_head_kernel(
    const uint16_t* __restrict__ hidden, int64_t n_rows, int H, int64_t ld_h, const uint16_t* __restrict__ w,
    float bias, const int32_t* __restrict__ rows, const int32_t* __restrict__ out_index, int64_t M,
    const int64_t* __restrict__ m_actual, float* __restrict__ out, int32_t* status) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t m_eff = m_actual ? min(M, *m_actual) : M;
    const int64_t step = (int64_t)gridDim.x * kVhWaves * kRows;
    for (int64_t t0 = ((int64_t)blockIdx.x * kVhWaves + wave) * kRows; t0 < m_eff; t0 += step) {
    // lane r < kRows looks up row r (the last row again beyond the end: read, not written)
    const int64_t mine = min(t0 + lane % kRows, m_eff - 1);
    const int64_t want = rows ? (int64_t)rows[mine] : mine;
    const bool bad = want < 0 || want >= n_rows;
    const int64_t row = min(max(want, (int64_t)0), n_rows - 1);
    const vh_chunk* src[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const uint32_t lo = __builtin_amdgcn_readlane((int)row, r), hi = __builtin_amdgcn_readlane((int)(row >> 32), r);
        src[r] = reinterpret_cast<const vh_chunk*>(hidden + (int64_t)((uint64_t)hi << 32 | lo) * ld_h);
    }
    float acc[kRows][4];
#pragma unroll
    for (int r = 0; r < kRows; ++r)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[r][e] = 0.f;
    const int chunks = H / 8;                                   // 16-byte pieces per row
#pragma unroll 2
    for (int c = lane; c < chunks; c += kWave) {
        vh_chunk x[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r) x[r] = __builtin_nontemporal_load(src[r] + c);
        const vh_weights k = *(reinterpret_cast<const vh_weights*>(w) + c);
#pragma unroll
        for (int r = 0; r < kRows; ++r)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc[r][2 * (e & 1)] = fmaf(__uint_as_float(x[r][e] << 16), __uint_as_float(k[e] << 16),
                                           acc[r][2 * (e & 1)]);
                acc[r][2 * (e & 1) + 1] = fmaf(__uint_as_float(x[r][e] & 0xFFFF0000u),
                                               __uint_as_float(k[e] & 0xFFFF0000u), acc[r][2 * (e & 1) + 1]);
            }
    }
    float total = 0.f;                                          // lane r: row r's sum
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const float s = wave_prefix((acc[r][0] + acc[r][1]) + (acc[r][2] + acc[r][3]));
        const float sum = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s), kWave - 1));   // (by all lanes, whoever keeps it)
        total = lane == r ? sum : total;
    }
    if (lane < kRows && t0 + lane < m_eff) {
        const int64_t o = out_index ? (int64_t)out_index[t0 + lane] : t0 + lane;
        if (bad) set_status(status, TPPO_STATUS_BAD_ROW);
        out[o] = bad ? __builtin_nanf("") : total + bias;
    }
    }
}

}  // namespace tppo

extern "C" int tppo_value_head(const void* hidden, int64_t n_rows, int64_t H, int64_t ld_hidden,
                               const void* w_value, float bias, tppo_dtype dt, const int32_t* rows,
                               const int32_t* out_index, int64_t M, const int64_t* m_actual, float* v_out,
                               int32_t* status, void* stream) {
    using namespace tppo;
    if (dt != TPPO_BF16) return TPPO_ERR_DTYPE;
    if (M < 0 || H <= 0 || n_rows < 0 || H > kVhMaxH || ld_hidden < H) return TPPO_ERR_SIZE;
    if (M == 0) return TPPO_OK;
    if (n_rows == 0) return TPPO_ERR_SIZE;
    if (!hidden || !w_value || !v_out) return TPPO_ERR_NULL;
    if (H % 8 != 0 || ld_hidden % 8 != 0 || !is_aligned(hidden, 16)) return TPPO_ERR_PARAM;
    // Two rows per wavefront up to three workgroups of eight rows to a CU, where their time jumps; four beyond.  Measured at
    // H = 5120, two / four, us: 2000 rows 6.8 / 10.1, 6016 rows 11.7 / 12.4, 6144 rows 11.9 / 12.3, 6152 rows 13.7 / 12.4,
    // 7168 rows 15.2 / 13.6, 8000 rows 15.6 / 14.8; the same line at H = 2048, 3584 and 8192.
    auto go = [&](auto kernel, int per_wave) {
        const int64_t per_group = (int64_t)kVhWaves * per_wave;
        const int64_t want = (M + per_group - 1) / per_group;
        hipLaunchKernelGGL(kernel, dim3((unsigned)(want < kVhMaxGroups ? want : kVhMaxGroups)), dim3(kVhThreads), 0,
                           static_cast<hipStream_t>(stream), static_cast<const uint16_t*>(hidden), n_rows, (int)H, ld_hidden,
                           static_cast<const uint16_t*>(w_value), bias, rows, out_index, M, m_actual, v_out, status);
    };
    if (M > kVhFewRows) go(value_head_kernel<4>, 4);
    else go(value_head_kernel<2>, 2);
    return launch_result();
}
