// tppo_token_logprobs_backward: derivatives of the kept tokens' log-probs with
// respect to the hidden rows and the head matrix, without keeping logits from
// the forward pass.  With z = W h, logp = z[target] - lse:
//     dz[t, v] = g_t * ([v == target_t] - exp(z[t, v] - lse_t))
//     d/dh_t   = sum_v dz[t, v] W[v, :]          (dZ  . W)
//     d/dW_v   = sum_t dz[t, v] h_t              (dZ^T . Hid)
// The logits are recomputed tile by tile with the forward kernel's sweep, whose
// epilogue here turns each finished tile into dz and writes it as bf16 for a
// chunk of tokens at a time; the two products are the same sweep again with a
// plain store epilogue.  W in the first and dZ in the second have K as their row
// index and are read that way (K-major operands, head_tile.h); only the gathered
// Hid^T, H x tokens, is made by a tiled transpose.
#include "head_tile.h"

namespace tppo {

// two fp32 -> two bf16 in one instruction, round to nearest even
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{lo, hi}), bf16x2));
}

// Epilogue 1: a finished tile of logits (vocabulary x tokens) becomes
// dz, row t of `out`, which is ld_out wide and lies in blocks (head_tile.h,
// block_at).  A lane owns one token column per block, and of each block of 16
// vocabulary entries the 4 of its lane group; two blocks' worth is
// exchanged between the four lane groups of a token so that each holds 8
// consecutive entries: 16-byte stores, 64 bytes of a block's row side by side.
// This runs once per tile with every matrix core idle, so its instructions count:
// per entry one fma, one exp2, one multiply, half a conversion, half a swap; the
// sampled token and the ragged last tile are rare branches.  Measured: 16414
// tokens, H = 1024, V = 32000, the whole backward call 3.33 -> 3.21 ms against
// per-entry selects, rounding in integer steps and 8-byte stores.  (Non-temporal
// stores: 3 % faster at H = 512, as fast there, 4 % slower at 4096 tokens, V = 152064, 2 % at H = 3584.)
template <class C>
struct DzEpilogue {
    static constexpr bool kPrefetch = false, kDealt = true;
    float lse2[C::kTB], g[C::kTB];
    int tgt[C::kTB];

    __device__ __forceinline__ void init(const HeadParams& p, int64_t tok0, int64_t m_eff, int wt, int lane) {
#pragma unroll
        for (int tb = 0; tb < C::kTB; ++tb) {
            const int64_t t = tok0 + wt * C::kWaveT + tb * C::kMI + (lane % C::kMI);
            lse2[tb] = 0.f;
            g[tb] = 0.f;
            tgt[tb] = -1;
            if (t < m_eff) {
                const int64_t i = p.aux_index ? (int64_t)p.aux_index[t] : t;
                lse2[tb] = p.aux0[i] * kLog2e;
                g[tb] = p.aux1[i];
                tgt[tb] = p.sel_targets[t];
            }
        }
    }

    __device__ __forceinline__ void fold(typename C::Acc (&acc)[C::kVB][C::kTB], const HeadParams& p, const Task& task,
                                         int64_t tok0, int64_t m_eff, int v0, int wv, int wt, int lane) {
        constexpr int kVB = C::kVB, kTB = C::kTB, kE = C::kAccElems;
        const int grp = lane / C::kMI, v_wave = v0 + wv * C::kWaveV;
        const int stored = task.v_end == p.V ? (int)p.out_cols : task.v_end;    // columns up to here are this task's
        char* out = static_cast<char*>(p.out);
        if (v0 + C::kTileV > task.v_end) {                          // ragged last tile: no entry there, dz = 0
            int left = task.v_end - v_wave - C::row_in_wave(0, 0, grp);
#pragma unroll
            for (int vb = 0; vb < kVB; ++vb) {
                asm volatile("" : "+v"(left));                      // (one block's masks at a time: the scalar registers are full)
#pragma unroll
                for (int tb = 0; tb < kTB; ++tb)
#pragma unroll
                    for (int e = 0; e < kE; ++e)
                        if (C::row_in_wave(vb, e, 0) >= left) acc[vb][tb][e] = -INFINITY;
            }
        }
#pragma unroll
        for (int tb = 0; tb < kTB; ++tb) {
            __builtin_amdgcn_sched_barrier(0);                      // (one token column at a time: the registers are full)
#pragma unroll
            for (int vb = 0; vb < kVB; ++vb)
#pragma unroll
                for (int e = 0; e < kE; ++e)
                    acc[vb][tb][e] = __builtin_amdgcn_exp2f(fmaf(acc[vb][tb][e], kLog2e, -lse2[tb]));
            const int d = tgt[tb] - v_wave - 4 * grp;               // the sampled token's entry: in few waves
            if (__any(d >= 0 && d < C::kWaveV && (d & 12) == 0)) {
#pragma unroll
                for (int vb = 0; vb < kVB; ++vb)
#pragma unroll
                    for (int e = 0; e < kE; ++e) acc[vb][tb][e] -= d == vb * C::kMI + e ? 1.f : 0.f;
            }
            const int64_t t = tok0 + wt * C::kWaveT + tb * C::kMI + (lane % C::kMI);
            char* row = out + C::block_at(t, v_wave, p.ld_out);
#pragma unroll
            for (int vb = 0; vb < kVB; vb += 2) {
                uint32_t a[2], b[2];                                // groups 0-3 of block vb, of block vb + 1
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    a[j] = pack_bf16(-g[tb] * acc[vb][tb][2 * j], -g[tb] * acc[vb][tb][2 * j + 1]);
                    b[j] = pack_bf16(-g[tb] * acc[vb + 1][tb][2 * j], -g[tb] * acc[vb + 1][tb][2 * j + 1]);
                    // a0 a1 a2 a3 | b0 b1 b2 b3  ->  a0 a1 b0 b1 | a2 a3 b2 b3  ->  a0 a2 b0 b2 | a1 a3 b1 b3
                    const auto half = __builtin_amdgcn_permlane32_swap(a[j], b[j], false, false);
                    const auto quarter = __builtin_amdgcn_permlane16_swap(half[0], half[1], false, false);
                    a[j] = quarter[0];
                    b[j] = quarter[1];
                }
                const int v = v_wave + vb * C::kMI + grp * 8;
                if (t < m_eff && v < stored)
                    *reinterpret_cast<uint4*>(row + C::block_at(0, vb * C::kMI + grp * 8, 0)) = make_uint4(a[0], a[1], b[0], b[1]);
            }
        }
#pragma unroll
        for (int vb = 0; vb < C::kVB; ++vb)
#pragma unroll
            for (int tb = 0; tb < C::kTB; ++tb)
#pragma unroll
                for (int e = 0; e < C::kAccElems; ++e) acc[vb][tb][e] = 0.f;
    }

    __device__ __forceinline__ void finish(const HeadParams&, float*, const Task&, int64_t, int64_t, int, int, int, int) {}
};

// The same in large tiles up to H = kPrefetchH, with W's lines brought ahead.
template <class C>
struct DzAheadEpilogue : DzEpilogue<C> {
    static constexpr bool kPrefetch = true;
};

// Epilogue 2: plain store of the fp32 tile, out[t, v] (+)= acc -- the sweep as the
// product out[T, V] = tokens[T, K] . w_role[V, K]^T.  A tile that holds one chunk of the contraction goes
// whole into its place among the partial tiles.
template <class C>
struct StoreEpilogue {
    static constexpr bool kPrefetch = false, kDealt = false;
    __device__ __forceinline__ void init(const HeadParams&, int64_t, int64_t, int, int) {}

    __device__ __forceinline__ void fold(typename C::Acc (&acc)[C::kVB][C::kTB], const HeadParams& p, const Task& task,
                                         int64_t tok0, int64_t m_eff, int v_tile, int wv, int wt, int lane) {
        const bool partial = task.rest && p.k_chunks > 1;
        const int v_lane = (partial ? 0 : v_tile) + wv * C::kWaveV + (lane / C::kMI) * 4;
        float* out = partial ? p.part_rest + (int64_t)task.part * (C::kTileV * C::kTileT) - tok0 * C::kTileV
                             : static_cast<float*>(p.out);
        const int64_t ld_out = partial ? C::kTileV : p.ld_out, out_cols = p.out_cols - (partial ? v_tile : 0);
        const bool accumulate = p.accumulate && !partial;
#pragma unroll
        for (int tb = 0; tb < C::kTB; ++tb) {
            const int64_t t = tok0 + wt * C::kWaveT + tb * C::kMI + (lane % C::kMI);
            if (t < m_eff) {
                float* row = out + t * ld_out;
#pragma unroll
                for (int vb = 0; vb < C::kVB; ++vb) {
                        const int v0 = v_lane + vb * C::kMI;
                        if (v0 < out_cols) {
                            float4 val = make_float4(acc[vb][tb][0], acc[vb][tb][1], acc[vb][tb][2], acc[vb][tb][3]);
                            float4* dst = reinterpret_cast<float4*>(row + v0);
                            if (accumulate) {
                                const float4 old = *dst;
                                val.x += old.x; val.y += old.y; val.z += old.z; val.w += old.w;
                            }
                            *dst = val;
                        }
                    }
            }
        }
#pragma unroll
        for (int vb = 0; vb < C::kVB; ++vb)
#pragma unroll
            for (int tb = 0; tb < C::kTB; ++tb)
#pragma unroll
                for (int e = 0; e < C::kAccElems; ++e) acc[vb][tb][e] = 0.f;
    }

    __device__ __forceinline__ void finish(const HeadParams&, float*, const Task&, int64_t, int64_t, int, int, int, int) {}
};

// The output tiles whose contraction was cut: out (+)= the sum of their partial tiles, in chunk order.  One
// workgroup per 4 rows of a tile, a float4 per thread (16 rows, four to a thread: 10.0 us for 4 tiles in 15 chunks; now 8.2 for
// 4 in 32).
constexpr int kSumRows = 4;                        // one for each wavefront, a float4 for each lane
static_assert(kTile % kSumRows == 0 && kTile == 4 * kWave, "a workgroup covers whole rows of a tile");
__global__ __launch_bounds__(kSumRows * kWave) void sum_chunks_kernel(HeadParams p) {
    const int id = blockIdx.x / (kTile / kSumRows), r0 = blockIdx.x % (kTile / kSumRows) * kSumRows;
    const Task task = task_at<true>(p, p.first_tasks + id, 1);
    const int64_t t0 = (int64_t)task.row * kTile + r0;
    const int v = (threadIdx.x & 63) * 4, r = threadIdx.x >> 6;
    const int64_t v0 = (int64_t)task.col * kTile + v;
    if (v0 >= p.out_cols || t0 + r >= p.M) return;
    float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
    const float* at = p.part_rest + (int64_t)id * (kTile * kTile) + (r0 + r) * kTile + v;
#pragma unroll 4
    for (int c = 0; c < p.k_chunks; ++c) {
        const float4 x = *reinterpret_cast<const float4*>(at + (int64_t)c * p.rest_tasks * (kTile * kTile));
        sum.x += x.x; sum.y += x.y; sum.z += x.z; sum.w += x.w;
    }
    float4* dst = reinterpret_cast<float4*>(static_cast<float*>(p.out) + (t0 + r) * p.ld_out + v0);
    if (p.accumulate) {
        const float4 old = *dst;
        sum.x += old.x; sum.y += old.y; sum.z += old.z; sum.w += old.w;
    }
    *dst = sum;
}

// dst[c, r] = src[index ? index[r] : r, c] for r < rows (0 for rows <= r < the
// next multiple of 64), c < cols; 2-byte elements, 64 x 64 tiles through LDS,
// 32-byte accesses on both sides.  cols % 64 == 0; rows of src and dst 16-byte aligned.
constexpr int kTrTile = 64, kTrThreads = 256;
__global__ __launch_bounds__(kTrThreads) void transpose_bf16_kernel(
    const uint16_t* __restrict__ src, int64_t rows, int64_t cols, int64_t ld_src,
    const int32_t* __restrict__ index, int64_t index_rows, uint16_t* __restrict__ dst, int64_t ld_dst) {
    __shared__ uint16_t tile[kTrTile][kTrTile + 2];
    const int64_t r0 = (int64_t)blockIdx.x * kTrTile, c0 = (int64_t)blockIdx.y * kTrTile;
    const int tid = threadIdx.x, i = tid >> 2, part = (tid & 3) * 16;
    {
        const int64_t r = r0 + i;
        uint4 a = make_uint4(0, 0, 0, 0), b = a;
        if (r < rows) {
            int64_t sr = index ? (int64_t)index[r] : r;
            sr = min(max(sr, (int64_t)0), index_rows - 1);
            const uint4* s = reinterpret_cast<const uint4*>(src + sr * ld_src + c0 + part);
            a = s[0];
            b = s[1];
        }
        const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            tile[i][part + 2 * j] = (uint16_t)(w[j] & 0xFFFFu);
            tile[i][part + 2 * j + 1] = (uint16_t)(w[j] >> 16);
        }
    }
    __syncthreads();
    {
        const int64_t c = c0 + i;                          // dst row
        uint32_t w[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            w[j] = (uint32_t)tile[part + 2 * j][i] | ((uint32_t)tile[part + 2 * j + 1][i] << 16);
        if (c < cols) {
            uint4* d = reinterpret_cast<uint4*>(dst + c * ld_dst + r0 + part);
            d[0] = make_uint4(w[0], w[1], w[2], w[3]);
            d[1] = make_uint4(w[4], w[5], w[6], w[7]);
        }
    }
}

static int launch_transpose(const uint16_t* src, int64_t rows, int64_t cols, int64_t ld_src, const int32_t* index,
                            int64_t index_rows, uint16_t* dst, int64_t ld_dst, hipStream_t s) {
    const dim3 grid((unsigned)((rows + kTrTile - 1) / kTrTile), (unsigned)(cols / kTrTile));
    hipLaunchKernelGGL(transpose_bf16_kernel, grid, dim3(kTrThreads), 0, s, src, rows, cols, ld_src, index,
                       index_rows, dst, ld_dst);
    return launch_result();
}

using BwdCfg = HeadCfg<uint16_t, false>;

// out[M, N] (+)= tokens[M, K] . w_role[N, K]^T, one of the two K-major, divided by plan_bwd_product.
// Transposing W and dZ first (both operands read along K, b128 fragments) moves 2 x 2 bytes per entry of both through
// memory, 7 to 13 % of the call, and needs their room; the K-major sweep itself is 2 to 6 % slower (twice the LDS
// instructions for one operand).  Whole call, transposes -> now: 16414 tokens, H = 1024, V = 32000: 3.28 -> 2.91 ms; 3514
// tokens, H = 5120, V = 152064: 14.38 -> 13.69 ms.
template <int KMAJOR>
static int launch_product(HeadParams& p, void* arrivals, hipStream_t s) {
    if (launch_sweep<HeadCfg<uint16_t, false, false, KMAJOR>, StoreEpilogue>(p, p.k_tiles > kAlignStages ? arrivals : nullptr, s) !=
        TPPO_OK)
        return TPPO_ERR_LAUNCH;
    if (p.k_chunks == 1) return TPPO_OK;
    hipLaunchKernelGGL(sum_chunks_kernel, dim3((unsigned)(p.rest_tasks * (kTile / kSumRows))), dim3(kSumRows * kWave), 0, s, p);
    return launch_result();
}

constexpr int64_t kBwdChunkDefault = 98304, kBwdChunkMax = 98304;

struct BwdLayout {
    int64_t v_pad, chunk;              // vocabulary padded to 64; tokens per chunk (multiple of 256)
    size_t off_dz, off_hidt, off_arrivals, off_part, total;
};

// Room for the partial tiles of a cut contraction: 512 of them, two rounds, at most.  The least that a call is content with is
// as much as dZ takes; what a workspace has beyond that is used as well.
constexpr size_t kPartBytes = (size_t)512 * kTile * kTile * sizeof(float);

static BwdLayout bwd_layout(int64_t H, int64_t V, int64_t chunk) {
    BwdLayout L;
    L.v_pad = (V + 63) / 64 * 64;
    L.chunk = chunk;
    size_t o = 0;
    const size_t dz = round_up((size_t)chunk * L.v_pad * 2, 256);
    L.off_dz = o;       o += dz;                                               // dZ    [chunk, v_pad] in blocks
    L.off_hidt = o;     o += round_up((size_t)H * chunk * 2, 256);             // Hid^T [H, chunk]
    L.off_arrivals = o; o += arrivals_bytes(chunk > V ? chunk : V);
    L.off_part = o;     o += dz < kPartBytes ? dz : kPartBytes;
    L.total = o;
    return L;
}

// The two products of `mc` tokens: 0, dZ . W for grad_hidden; 1, dZ^T . Hid for grad_w.
static void plan_bwd_product(HeadParams& p, int product, int64_t mc, int64_t H, int64_t V, void* part, size_t part_bytes) {
    p.k_tiles = (int)(((product == 0 ? V : mc) + BwdCfg::kBK - 1) / BwdCfg::kBK);
    plan_product(p, product == 0 ? mc : V, H, part, part_bytes);
}

// What the products of the call's chunks cut into, given room: with as much, or more, they are divided one and the same way.
static size_t wanted_part_bytes(int64_t M, int64_t chunk, int64_t H, int64_t V) {
    size_t most = 0;
    for (int64_t mc : {std::min(M, chunk), M % chunk})
        for (int product = 0; product < 2 && mc > 0; ++product) {
            HeadParams p = {};
            plan_bwd_product(p, product, mc, H, V, nullptr, kPartBytes);
            if (p.k_chunks > 1) most = std::max(most, (size_t)p.k_chunks * p.rest_tasks * kTile * kTile * sizeof(float));
        }
    return most;
}

}  // namespace tppo

extern "C" size_t tppo_token_logprobs_backward_workspace_bytes(int64_t M, int64_t H, int64_t V, tppo_dtype dt) {
    using namespace tppo;
    if (M <= 0 || H <= 0 || V <= 0 || dt != TPPO_BF16) return 256;
    const int64_t m_round = (M + 255) / 256 * 256;
    const BwdLayout L = bwd_layout(H, V, m_round < kBwdChunkDefault ? m_round : kBwdChunkDefault);
    return std::max(L.total, L.off_part + wanted_part_bytes(M, L.chunk, H, V));
}

extern "C" int tppo_token_logprobs_backward(const void* hidden, int64_t n_rows, int64_t H, int64_t ld_hidden,
                                            const void* w_head, int64_t V, int64_t ld_w, tppo_dtype dt,
                                            const int32_t* sel_rows, const int32_t* sel_targets, int64_t M,
                                            const float* lse, const float* grad_logp, const int32_t* in_index,
                                            float* grad_hidden, float* grad_w, int32_t accumulate_w,
                                            void* workspace, size_t workspace_bytes, int32_t* status,
                                            void* stream) {
    using namespace tppo;
    (void)status;
    if (dt != TPPO_BF16) return TPPO_ERR_DTYPE;
    if (M < 0 || H <= 0 || V <= 0 || n_rows <= 0 || M > INT32_MAX || V > INT32_MAX - 4096 || H > INT32_MAX)
        return TPPO_ERR_SIZE;
    if (ld_hidden < H || ld_w < H) return TPPO_ERR_SIZE;
    if (H % 64 != 0 || ld_hidden % 8 != 0 || ld_w % 8 != 0 || !is_aligned(hidden, 16) || !is_aligned(w_head, 16))
        return TPPO_ERR_PARAM;
    if (M == 0 || (!grad_hidden && !grad_w)) return TPPO_OK;
    if (!hidden || !w_head || !sel_rows || !sel_targets || !lse || !grad_logp) return TPPO_ERR_NULL;
    if ((grad_hidden && !is_aligned(grad_hidden, 16)) || (grad_w && !is_aligned(grad_w, 16))) return TPPO_ERR_PARAM;
    if (!workspace || !is_aligned(workspace, 256)) return TPPO_ERR_WORKSPACE;
    // the largest chunk (multiple of 256 tokens) the workspace holds
    const int64_t m_round = (M + 255) / 256 * 256;
    int64_t chunk = m_round < kBwdChunkMax ? m_round : kBwdChunkMax;
    while (chunk >= 256 && bwd_layout(H, V, chunk).total > workspace_bytes) chunk -= 256;
    if (chunk < 256) return TPPO_ERR_WORKSPACE;
    const BwdLayout L = bwd_layout(H, V, chunk);
    char* ws = static_cast<char*>(workspace);
    uint16_t* dz = reinterpret_cast<uint16_t*>(ws + L.off_dz);
    uint16_t* hidt = reinterpret_cast<uint16_t*>(ws + L.off_hidt);
    void *arrivals = ws + L.off_arrivals, *part = ws + L.off_part;
    const size_t part_bytes = std::min(kPartBytes, workspace_bytes - L.off_part);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint16_t* hid = static_cast<const uint16_t*>(hidden);
    const uint16_t* w = static_cast<const uint16_t*>(w_head);

    for (int64_t m0 = 0; m0 < M; m0 += chunk) {
        const int64_t mc = M - m0 < chunk ? M - m0 : chunk;
        const int64_t m_pad = (mc + 63) / 64 * 64;
        // 1. dZ[mc, v_pad] (bf16): logits recomputed, softmax derivative applied
        HeadParams p = {};
        p.hidden = hid; p.n_rows = n_rows; p.ld_h = ld_hidden;
        p.w = w; p.ld_w = ld_w; p.H = (int)H; p.k_tiles = (int)(H / BwdCfg::kBK);
        p.sel_rows = sel_rows + m0;
        p.sel_targets = sel_targets + m0;
        p.aux0 = in_index ? lse : lse + m0;
        p.aux1 = in_index ? grad_logp : grad_logp + m0;
        p.aux_index = in_index ? in_index + m0 : nullptr;
        p.out = dz; p.ld_out = L.v_pad; p.out_cols = L.v_pad;
        const bool small = plan_small(p, mc, V, plan_sweep(p, mc, V));
        const int narrow = plan_narrow(p, mc, V, small);
        if ((narrow            ? launch_narrow<false, DzEpilogue>(narrow, p, s)
             : small           ? launch_sweep<SmallShape, DzEpilogue>(p, arrivals, s)
             : H <= kPrefetchH ? launch_sweep<BwdCfg, DzAheadEpilogue>(p, arrivals, s)
                               : launch_sweep<BwdCfg, DzEpilogue>(p, arrivals, s)) != TPPO_OK)
            return TPPO_ERR_LAUNCH;
        // 2. grad_hidden[m0 + t, :] = dZ[t, :] . W   (token role: dZ rows; W role: columns of W; K = v_pad)
        if (grad_hidden) {
            HeadParams q = {};
            q.hidden = dz; q.n_rows = mc; q.ld_h = L.v_pad;
            q.w = w; q.ld_w = ld_w; q.H = (int)L.v_pad;
            q.km_rows = (int)V; q.km_cols = (int)H;
            q.out = grad_hidden + m0 * H; q.ld_out = H; q.out_cols = H;
            plan_bwd_product(q, 0, mc, H, V, part, part_bytes);
            if (launch_product<1>(q, arrivals, s) != TPPO_OK) return TPPO_ERR_LAUNCH;
        }
        // 3. grad_w[v, :] (+)= dZ^T[v, :] . Hid   (token role: columns of dZ; W role: rows of Hid^T; K = m_pad)
        if (grad_w) {
            if (launch_transpose(hid, mc, H, ld_hidden, sel_rows + m0, n_rows, hidt, m_pad, s) != TPPO_OK)
                return TPPO_ERR_LAUNCH;
            HeadParams q = {};
            q.hidden = dz; q.n_rows = mc; q.ld_h = L.v_pad;
            q.w = hidt; q.ld_w = m_pad; q.H = (int)m_pad;
            q.km_rows = (int)mc; q.km_cols = (int)L.v_pad;
            q.out = grad_w; q.ld_out = H; q.out_cols = H;
            q.accumulate = (m0 > 0 || accumulate_w) ? 1 : 0;
            plan_bwd_product(q, 1, mc, H, V, part, part_bytes);
            if (launch_product<2>(q, arrivals, s) != TPPO_OK) return TPPO_ERR_LAUNCH;
        }
    }
    return TPPO_OK;
}
