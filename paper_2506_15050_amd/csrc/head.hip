// tppo_token_logprobs: log pi_theta(a_t|s_t) of the kept tokens -- the LM head
// W_head h fused with log-softmax and the gather of the sampled token's logit
// (the quantity inside the ratio of Eq. (ppoloss)); logits never reach memory.
//
// Matrix-core path.  The logits of a 256-token x 256-vocabulary tile (64 x 128 in
// calls too small for those, in fp32 and for long ragged rows; 64 to 192 x 256 in between) are accumulated with
// v_mfma_f32_16x16x32_bf16 or 16x16x4_f32 (head_tile.h).
// The MFMA "row" operand is the W tile and the "column" operand the gathered
// hidden rows, so the accumulators a lane holds for one block all belong to ONE
// token (column lane % 16) and to different vocabulary entries: the running
// maximum, the running sum of exponentials and the target logit of a token
// live in that lane's registers across all vocabulary tiles of the sweep, with
// no cross-lane traffic until the very end.  The work is (token tiles) x
// (vocabulary splits), dealt out by the schedule of head_tile.h; each pair
// sweeps its share of vocabulary tiles and writes one (max, sumexp, target
// logit) triple per token; a small kernel merges the splits into logp and lse.
//
// Both operands are K-contiguous in memory ([V,H] and [rows,H]), which is the
// layout the MFMA wants for both, so tiles are staged into LDS as 16-byte
// chunks with an XOR swizzle of the chunk index (conflict-free ds_read_b128)
// and read back as operand fragments directly.
#include "head_tile.h"

namespace tppo {

// ------------------------------------------------------------------ generic
// One workgroup per kept token, one wavefront per vocabulary row at a time,
// fp32 FMA: every token reads all of W, so it runs at a hundredth of the matrix
// cores' rate.  Serves what the tiled kernel's 16-byte transfers cannot address:
// base pointers or leading dimensions that are not multiples of 16 bytes where
// the workspace has no room for aligned copies, and fp32 calls without a workspace.
constexpr int kGenThreads = 256;
constexpr int kGenMaxH = 16320;               // the hidden row (fp32) and 48 bytes of partial results share 64 KiB of LDS

__device__ __forceinline__ float load_as_float(const float* p, int64_t i) { return p[i]; }
__device__ __forceinline__ float load_as_float(const uint16_t* p, int64_t i) {
    return __uint_as_float((unsigned)p[i] << 16);
}

template <typename T>
__global__ __launch_bounds__(kGenThreads) void head_generic_kernel(
    const T* __restrict__ hidden, int64_t n_rows, int H, int64_t ld_h, const T* __restrict__ w,
    int V, int64_t ld_w, const int32_t* __restrict__ sel_rows,
    const int32_t* __restrict__ sel_targets, int64_t M, const int64_t* __restrict__ m_actual,
    const int32_t* __restrict__ out_index, float* __restrict__ logp, float* __restrict__ lse,
    int32_t* status) {
    extern __shared__ float s_h[];
    __shared__ float s_part[3][kGenThreads / kWave];
    const int64_t m = blockIdx.x;
    const int64_t m_eff = m_actual ? min(M, *m_actual) : M;
    if (m >= m_eff) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t row = sel_rows[m];
    const int tgt = sel_targets[m];
    const int64_t o = out_index ? (int64_t)out_index[m] : m;
    const bool bad_row = row < 0 || row >= n_rows, bad_tgt = tgt < 0 || tgt >= V;
    if (bad_row || bad_tgt) {
        if (tid == 0) {
            set_status(status, bad_row ? TPPO_STATUS_BAD_ROW : TPPO_STATUS_BAD_TARGET);
            logp[o] = __builtin_nanf("");
            if (lse) lse[o] = __builtin_nanf("");
        }
        return;
    }
    for (int k = tid; k < H; k += kGenThreads) s_h[k] = load_as_float(hidden, row * ld_h + k);
    __syncthreads();
    float mx = -INFINITY, sum = 0.f, tz = 0.f;
    for (int v = wave; v < V; v += kGenThreads / kWave) {
        const T* wr = w + (int64_t)v * ld_w;
        float z = 0.f;
        for (int k = lane; k < H; k += kWave) z = fmaf(s_h[k], load_as_float(wr, k), z);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) z += __shfl_xor(z, off);
        const float mn = fmaxf(mx, z);
        sum = sum * expf(mx - mn) + expf(z - mn);
        mx = mn;
        if (v == tgt) tz = z;
    }
    if (lane == 0) {
        s_part[0][wave] = mx;
        s_part[1][wave] = sum;
        s_part[2][wave] = tz;
    }
    __syncthreads();
    if (tid == 0) {
        float gm = -INFINITY, gs = 0.f, gt = 0.f;
        for (int q = 0; q < kGenThreads / kWave; ++q) gm = fmaxf(gm, s_part[0][q]);
        for (int q = 0; q < kGenThreads / kWave; ++q) {
            if (s_part[1][q] > 0.f) gs += s_part[1][q] * expf(s_part[0][q] - gm);
            gt += s_part[2][q];
        }
        const float l = gm + logf(gs);
        logp[o] = gt - l;
        if (lse) lse[o] = l;
    }
}

// ------------------------------------------------------------------ MFMA path
// What a running maximum is held in: logits, or logits * log2(e) (head_tile.h, kLogitMax).
template <bool kLogitMax>
struct MaxUnits {
    static constexpr float kLeast = kLogitMax ? kLowest : kNegBig;
    __device__ static __forceinline__ float of(float z) { return kLogitMax ? z : z * kLog2e; }
    __device__ static __forceinline__ float log2_term(float z, float max) {
        return kLogitMax ? (z - max) * kLog2e : fmaf(z, kLog2e, -max);
    }
    __device__ static __forceinline__ float log2_ratio(float from, float to) {
        return kLogitMax ? (from - to) * kLog2e : from - to;
    }
};

// Per-lane running log-softmax state of the kTB token columns a lane owns, and
// the two steps that use it: folding a finished vocabulary tile, and
// the final merge across lane halves / waves.
template <class C>
struct LaneSoftmax {
    static constexpr bool kPrefetch = false, kDealt = false;
    typedef MaxUnits<C::kLogitMax> Units;
    float run_max[C::kTB], run_sum[C::kTB], tgt_logit[C::kTB];
    int tgt[C::kTB];

    __device__ __forceinline__ void init(const HeadParams& p, int64_t tok0, int64_t m_eff, int wt, int lane) {
#pragma unroll
        for (int tb = 0; tb < C::kTB; ++tb) {
            run_max[tb] = Units::kLeast;
            run_sum[tb] = 0.f;
            tgt_logit[tb] = 0.f;
            const int64_t t = tok0 + wt * C::kWaveT + tb * C::kMI + (lane % C::kMI);
            tgt[tb] = t < m_eff ? p.sel_targets[t] : -1;
        }
    }

    // acc holds logits: lane owns column lane % 16 of block tb; entry e of block vb
    // is vocabulary id v_wave + row_in_wave(vb, e, lane / 16).  Clears acc.
    __device__ __forceinline__ void fold(typename C::Acc (&acc)[C::kVB][C::kTB], const HeadParams&, const Task& task,
                                         int64_t, int64_t, int v0, int wv, int, int lane) {
        constexpr int kVB = C::kVB, kTB = C::kTB, kE = C::kAccElems;
        const int grp = lane / C::kMI;
        const int v_wave = v0 + wv * C::kWaveV;
        if (v0 + C::kTileV > task.v_end) {                          // ragged last tile: mask ids beyond the task's
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
            float mx0 = -INFINITY, mx1 = -INFINITY;
#pragma unroll
            for (int vb = 0; vb < kVB; ++vb)
#pragma unroll
                for (int e = 0; e < kE; e += 2) {
                    mx0 = fmaxf(mx0, acc[vb][tb][e]);
                    mx1 = fmaxf(mx1, acc[vb][tb][e + 1]);
                }
            const float new_max = fmaxf(run_max[tb], Units::of(fmaxf(mx0, mx1)));
            float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
#pragma unroll
            for (int vb = 0; vb < kVB; ++vb)
#pragma unroll
                for (int e = 0; e < kE; e += 4) {
                    s0 += __builtin_amdgcn_exp2f(Units::log2_term(acc[vb][tb][e], new_max));
                    s1 += __builtin_amdgcn_exp2f(Units::log2_term(acc[vb][tb][e + 1], new_max));
                    s2 += __builtin_amdgcn_exp2f(Units::log2_term(acc[vb][tb][e + 2], new_max));
                    s3 += __builtin_amdgcn_exp2f(Units::log2_term(acc[vb][tb][e + 3], new_max));
                }
            run_sum[tb] = fmaf(run_sum[tb], __builtin_amdgcn_exp2f(Units::log2_ratio(run_max[tb], new_max)), (s0 + s1) + (s2 + s3));
            run_max[tb] = new_max;
        }
        // target logit: rare (a lane owns kVB * kAccElems of V ids per tile), so only
        // waves in which some lane hits take the register-select path.  Row r of
        // a block belongs to lane group (r / 4) % kGroups, element (r / (4 kGroups)) * 4 + r % 4.
        const int in_tile = min(C::kWaveV, task.v_end - v_wave);    // (a sampled id beyond it is another task's)
        bool hit = false;
#pragma unroll
        for (int tb = 0; tb < kTB; ++tb) {
            const int d = tgt[tb] - v_wave;
            hit |= d >= 0 && d < in_tile && ((d >> 2) % C::kGroups) == grp;
        }
        if (__any(hit)) {
#pragma unroll
            for (int tb = 0; tb < kTB; ++tb) {
                const int d = tgt[tb] - v_wave;
                if (d >= 0 && d < in_tile && ((d >> 2) % C::kGroups) == grp) {
                    const int vb_t = d / C::kMI, r = d % C::kMI;
                    const int e_t = (r / (4 * C::kGroups)) * 4 + (r & 3);
                    float z = 0.f;
#pragma unroll
                    for (int vb = 0; vb < kVB; ++vb)
#pragma unroll
                        for (int e = 0; e < kE; ++e) z = (vb == vb_t && e == e_t) ? acc[vb][tb][e] : z;
                    tgt_logit[tb] += z;
                }
            }
        }
#pragma unroll
        for (int vb = 0; vb < kVB; ++vb)
#pragma unroll
            for (int tb = 0; tb < kTB; ++tb)
#pragma unroll
                for (int e = 0; e < kE; ++e) acc[vb][tb][e] = 0.f;
    }

    // Merge the lane groups (same token, different vocabulary rows), then
    // the kWavesV waves that share a token, and write the split's triple.
    // s_merge: LDS scratch [kWavesV][3][kTileT] floats, idle at this point.
    __device__ __forceinline__ void finish(const HeadParams& p, float* s_merge, const Task& task, int64_t tok0,
                                           int64_t m_eff, int wv, int wt, int lane, int tid) {
        constexpr int kTileT = C::kTileT;
#pragma unroll
        for (int off = C::kMI; off < 64; off <<= 1) {            // butterfly over the 64 / kMI lane groups
#pragma unroll
            for (int tb = 0; tb < C::kTB; ++tb) {
                const float om = __shfl_xor(run_max[tb], off), os = __shfl_xor(run_sum[tb], off);
                const float ot = __shfl_xor(tgt_logit[tb], off);
                const float nm = fmaxf(run_max[tb], om);
                run_sum[tb] = run_sum[tb] * __builtin_amdgcn_exp2f(Units::log2_ratio(run_max[tb], nm)) +
                              os * __builtin_amdgcn_exp2f(Units::log2_ratio(om, nm));
                run_max[tb] = nm;
                tgt_logit[tb] += ot;
            }
        }
        if (lane < C::kMI) {
#pragma unroll
            for (int tb = 0; tb < C::kTB; ++tb) {
                const int col = wt * C::kWaveT + tb * C::kMI + lane;
                s_merge[(wv * 3 + 0) * kTileT + col] = run_max[tb];
                s_merge[(wv * 3 + 1) * kTileT + col] = run_sum[tb];
                s_merge[(wv * 3 + 2) * kTileT + col] = tgt_logit[tb];
            }
        }
        __syncthreads();
        for (int col = tid; col < kTileT; col += C::kThreads) {
            const int64_t t = tok0 + col;
            if (t >= m_eff) continue;
            float gm = Units::kLeast, gs = 0.f, gt = 0.f;
#pragma unroll
            for (int q = 0; q < C::kWavesV; ++q) gm = fmaxf(gm, s_merge[(q * 3 + 0) * kTileT + col]);
#pragma unroll
            for (int q = 0; q < C::kWavesV; ++q) {
                gs += s_merge[(q * 3 + 1) * kTileT + col] *
                      __builtin_amdgcn_exp2f(Units::log2_ratio(s_merge[(q * 3 + 0) * kTileT + col], gm));
                gt += s_merge[(q * 3 + 2) * kTileT + col];
            }
            const Grid& g = task.rest ? p.rest : p.first;
            const int64_t tokens = (int64_t)g.rows * kTileT, plane = tokens * g.cols;
            float* out = (task.rest ? p.part_rest : p.part_first) + task.col * tokens + (t - (int64_t)g.row0 * kTileT);
            out[0] = gm;
            out[plane] = gs;
            out[2 * plane] = gt;
        }
    }
};

// Merge the columns' triples into logp and lse: 32 tokens per workgroup, 8 threads per token, each taking every
// eighth column (coalesced over the tokens), merged through LDS.  (One thread per token walking up to 64 columns
// twice took 20 us whatever the batch: a chain of dependent loads.)
struct Partials {
    const float *first, *rest;
    int64_t first_tokens;              // tokens of the first grid; the others belong to the rest
    int64_t first_stride, rest_stride; // tokens between two columns
    int first_cols, rest_cols;
};
constexpr int kMergeTokens = 32, kMergeLanes = 8;
template <bool kLogitMax>
__global__ __launch_bounds__(kMergeTokens* kMergeLanes) void head_combine_kernel(
    Partials q, int64_t M, const int64_t* __restrict__ m_actual,
    const int32_t* __restrict__ sel_rows, const int32_t* __restrict__ sel_targets, int64_t n_rows,
    int V, const int32_t* __restrict__ out_index, float* __restrict__ logp,
    float* __restrict__ lse, int32_t* status) {
    __shared__ float s_part[3][kMergeLanes][kMergeTokens];
    const int tok = threadIdx.x % kMergeTokens, sub = threadIdx.x / kMergeTokens;
    const int64_t m = (int64_t)blockIdx.x * kMergeTokens + tok;
    const int64_t m_eff = m_actual ? min(M, *m_actual) : M;
    typedef MaxUnits<kLogitMax> Units;
    float mx = Units::kLeast, sum = 0.f, tz = 0.f;
    // (what the end of the merge needs travels with the partials)
    int64_t o = m, row = 0;
    int tgt = 0;
    if (m < m_eff) {
        if (sub == 0) {
            if (out_index) o = out_index[m];
            row = sel_rows[m];
            tgt = sel_targets[m];
        }
        const bool rest = m >= q.first_tokens;
        const float* part = rest ? q.rest + (m - q.first_tokens) : q.first + m;
        const int64_t stride = rest ? q.rest_stride : q.first_stride;
        const int cols = rest ? q.rest_cols : q.first_cols;
        const int64_t plane = stride * cols;
#pragma unroll 4
        for (int c = sub; c < cols; c += kMergeLanes) {
            const float* at = part + c * stride;
            const float om = at[0], os = at[plane], ot = at[2 * plane];
            const float nm = fmaxf(mx, om);
            sum = sum * exp2f(Units::log2_ratio(mx, nm)) + os * exp2f(Units::log2_ratio(om, nm));
            mx = nm;
            tz += ot;
        }
    }
    s_part[0][sub][tok] = mx;
    s_part[1][sub][tok] = sum;
    s_part[2][sub][tok] = tz;
    __syncthreads();
    if (sub != 0 || m >= m_eff) return;
    const bool bad_row = row < 0 || row >= n_rows, bad_tgt = tgt < 0 || tgt >= V;
    if (bad_row || bad_tgt) {
        set_status(status, bad_row ? TPPO_STATUS_BAD_ROW : TPPO_STATUS_BAD_TARGET);
        logp[o] = __builtin_nanf("");
        if (lse) lse[o] = __builtin_nanf("");
        return;
    }
    float gm = Units::kLeast;
#pragma unroll
    for (int s = 0; s < kMergeLanes; ++s) gm = fmaxf(gm, s_part[0][s][tok]);
    float gs = 0.f, gt = 0.f;
#pragma unroll
    for (int s = 0; s < kMergeLanes; ++s) {
        gs += s_part[1][s][tok] * exp2f(Units::log2_ratio(s_part[0][s][tok], gm));
        gt += s_part[2][s][tok];
    }
    // The log-prob is put together before anything is rounded at the size of the logits: gt - lse would lose half an ulp of
    // them.  32000 logits of rms 1.4 and the sampled one at 8 to 12 / 30 to 35 / 60 to 65, rms error against 64 bits: 1.1e-7 /
    // 2.4e-9 / 0 in logits, 1.8e-7 / 2.5e-9 / 0 in log2, 9.5e-7 / 2.4e-9 / 0 by the one-token kernel; by gt - lse from log2
    // 4.2e-7 / 8e-7 / 1.7e-6, up to a third of them positive.
    if (kLogitMax) {
        const float log_sum = logf(gs);
        logp[o] = (gt - gm) - log_sum;
        if (lse) lse[o] = gm + log_sum;
    } else {
        const float log_sum = log2f(gs), l = (gm + log_sum) * kLn2, d = fmaf(gt, kLog2e, -gm);
        float lp = (d - log_sum) * kLn2;
        if (gt * kLog2e == gm) lp = logf(__builtin_amdgcn_exp2f(d) / gs);   // the largest: gs holds this very term, so 1 is 1
        else if (!isfinite(d)) lp = gt - l;                                 // (gt * log2(e) out of range)
        logp[o] = lp;
        if (lse) lse[o] = l;
    }
}

// Most partial triples a sweep of M tokens can write (plan_sweep: up to 4 columns in the whole rounds, kRestTasks
// tiles in the rest): grows with M, so a workspace sized for the largest batch serves every smaller one.
static int64_t most_triples(int64_t M) { return 4 * ((M + kTile - 1) / kTile * kTile) + kRestTasks * kTile; }

// Rows the tiled kernel cannot address (a row's start or length is no multiple of 16 bytes) are first copied, zero
// padded, to rows of whole chunks: dst[i] = src[index ? index[i] : i], 16 bytes per lane.  One read and one write
// of W and of the kept rows, against M reads of W by the generic kernel.
constexpr int kPackThreads = 256;
template <typename T>
__global__ __launch_bounds__(kPackThreads) void pack_rows_kernel(const T* __restrict__ src, int64_t n_src, int H,
                                                                 int64_t ld, const int32_t* __restrict__ index,
                                                                 int64_t rows, const int64_t* __restrict__ m_actual,
                                                                 T* __restrict__ dst, int chunks) {
    constexpr int kPer = 16 / sizeof(T);
    typedef T vec __attribute__((ext_vector_type(kPer), aligned(sizeof(T))));
    const int64_t n = (m_actual ? min(rows, *m_actual) : rows) * chunks, step = (int64_t)gridDim.x * kPackThreads;
    for (int64_t i = (int64_t)blockIdx.x * kPackThreads + threadIdx.x; i < n; i += step) {
        const int64_t r = i / chunks;
        const int k = (int)(i - r * chunks) * kPer;
        const int64_t from = index ? min(max((int64_t)index[r], (int64_t)0), n_src - 1) : r;
        const T* at = src + from * ld + k;
        vec x;
        if (k + kPer <= H) {
            x = *reinterpret_cast<const vec*>(at);
        } else {
#pragma unroll
            for (int e = 0; e < kPer; ++e) x[e] = k + e < H ? at[e] : (T)0;
        }
        *reinterpret_cast<vec*>(dst + r * (int64_t)chunks * kPer + k) = x;
    }
}

static size_t tiled_workspace(int64_t M) {
    return arrivals_bytes(M) + round_up((size_t)3 * (size_t)most_triples(M) * sizeof(float), 256);
}

static bool rows_addressable(const void* p, int64_t ld, int64_t H, size_t esz) {
    return is_aligned(p, 16) && (size_t)ld * esz % 16 == 0 && (size_t)H * esz % 16 == 0;
}

// aligned copies of W and of the kept rows, where the hidden size alone says they will be needed
static size_t packed_row_bytes(int64_t H, size_t esz) { return round_up((size_t)H * esz, 16); }
static size_t packed_bytes(int64_t M, int64_t H, int64_t V, size_t esz) {
    return round_up((size_t)(V + M) * packed_row_bytes(H, esz), 256);
}

template <typename T>
static int head_generic(const void* hidden, int64_t n_rows, int64_t H, int64_t ld_hidden, const void* w, int64_t V,
                        int64_t ld_w, const int32_t* sel_rows, const int32_t* sel_targets, int64_t M,
                        const int64_t* m_actual, const int32_t* out_index, float* logp, float* lse, int32_t* status,
                        hipStream_t s) {
    hipLaunchKernelGGL(head_generic_kernel<T>, dim3((unsigned)M), dim3(kGenThreads), (size_t)H * sizeof(float), s,
                       static_cast<const T*>(hidden), n_rows, (int)H, ld_hidden, static_cast<const T*>(w), (int)V, ld_w,
                       sel_rows, sel_targets, M, m_actual, out_index, logp, lse, status);
    return launch_result();
}

template <typename T>
static int head_tiled(HeadParams& p, int64_t M, int64_t V, const int32_t* out_index, float* logp, float* lse,
                      int64_t n_rows, const int32_t* sel_rows, bool matrix_only, void* workspace, int32_t* status, hipStream_t s) {
    typedef HeadCfg<T, false> Whole;
    typedef HeadCfg<T, true> Ragged;
    p.k_tiles = (p.H + Whole::kBK - 1) / Whole::kBK;
    const bool whole = p.H % Whole::kBK == 0;
    const bool small = plan_logprobs(p, M, V, sizeof(T) == 2, matrix_only);
    const int narrow = sizeof(T) == 2 ? plan_narrow(p, M, V, small) : 0;
    const int tile = narrow ? 64 * narrow : small ? SmallShape::kTileT : kTile;
    const int64_t first_tokens = (int64_t)p.first.rows * tile, rest_tokens = (int64_t)p.rest.rows * tile;
    const size_t room = arrivals_bytes(M);
    char* ws = static_cast<char*>(workspace);
    p.part_first = reinterpret_cast<float*>(ws + room);
    p.part_rest = p.part_first + 3 * first_tokens * p.first.cols;
    int rc = TPPO_ERR_LAUNCH;
    if (narrow) {
        rc = whole ? launch_narrow<false, LaneSoftmax>(narrow, p, s) : launch_narrow<true, LaneSoftmax>(narrow, p, s);
    } else if (small) {
        constexpr bool kFew = sizeof(T) == 4;                       // (HeadCfg: measured in fp32)
        if (kFew && p.n_tasks <= 2 * kSweepGroups)
            rc = whole ? launch_sweep<HeadCfg<T, false, true, 0, 4, kFew>, LaneSoftmax>(p, ws, s)
                       : launch_sweep<HeadCfg<T, true, true, 0, 4, kFew>, LaneSoftmax>(p, ws, s);
        else
            rc = whole ? launch_sweep<HeadCfg<T, false, true>, LaneSoftmax>(p, ws, s)
                       : launch_sweep<HeadCfg<T, true, true>, LaneSoftmax>(p, ws, s);
    } else if constexpr (sizeof(T) == 2) {
        typedef HeadCfg<T, false, false, 0, 4, false, true> Long;
        rc = !whole                     ? launch_sweep<Ragged, LaneSoftmax>(p, ws, s)
             : p.k_tiles >= kLongStages ? launch_sweep<Long, LaneSoftmax>(p, ws, s)
                                        : launch_sweep<Whole, LaneSoftmax>(p, ws, s);
    }
    if (rc != TPPO_OK) return rc;
    const Partials q = {p.part_first, p.part_rest, first_tokens, first_tokens, rest_tokens, p.first.cols, p.rest.cols};
    hipLaunchKernelGGL(head_combine_kernel<Whole::kLogitMax>, dim3((unsigned)((M + kMergeTokens - 1) / kMergeTokens)),
                       dim3(kMergeTokens * kMergeLanes), 0, s, q, M, p.m_actual, sel_rows, p.sel_targets, n_rows, (int)V,
                       out_index, logp, lse, status);
    return launch_result();
}

// Aligned copies first where the rows need them, then the tiled kernel.
template <typename T>
static int head_call(HeadParams& p, int64_t M, int64_t V, const int32_t* out_index, float* logp, float* lse,
                     void* workspace, size_t tiled_bytes, bool pack_h, bool pack_w, bool matrix_only, int32_t* status,
                     hipStream_t s) {
    const int64_t n_rows = p.n_rows;
    const int32_t* sel_rows = p.sel_rows;
    const int chunks = (int)(packed_row_bytes(p.H, sizeof(T)) / 16), per_row = chunks * (16 / (int)sizeof(T));
    T* copy = reinterpret_cast<T*>(static_cast<char*>(workspace) + tiled_bytes);
    auto groups = [&](int64_t rows) {
        const int64_t g = (rows * chunks + kPackThreads - 1) / kPackThreads;
        return dim3((unsigned)(g < 16384 ? g : 16384));
    };
    if (pack_w) {
        hipLaunchKernelGGL(pack_rows_kernel<T>, groups(V), dim3(kPackThreads), 0, s, static_cast<const T*>(p.w), V, p.H,
                           p.ld_w, (const int32_t*)nullptr, V, (const int64_t*)nullptr, copy, chunks);
        if (launch_result() != TPPO_OK) return TPPO_ERR_LAUNCH;
        p.w = copy;
        p.ld_w = per_row;
        copy += V * per_row;
    }
    if (pack_h) {
        hipLaunchKernelGGL(pack_rows_kernel<T>, groups(M), dim3(kPackThreads), 0, s, static_cast<const T*>(p.hidden),
                           p.n_rows, p.H, p.ld_h, p.sel_rows, M, p.m_actual, copy, chunks);
        if (launch_result() != TPPO_OK) return TPPO_ERR_LAUNCH;
        p.hidden = copy;
        p.ld_h = per_row;
        p.n_rows = M;
        p.sel_rows = nullptr;
    }
    if (pack_w || pack_h) p.H = per_row;                            // (zeros: they change no logit)
    return head_tiled<T>(p, M, V, out_index, logp, lse, n_rows, sel_rows, matrix_only, workspace, status, s);
}

}  // namespace tppo

extern "C" size_t tppo_token_logprobs_workspace_bytes(int64_t M, int64_t H, int64_t V,
                                                      tppo_dtype dt) {
    using namespace tppo;
    if (M <= 0 || V <= 0 || H <= 0 || (dt != TPPO_BF16 && dt != TPPO_F32)) return 256;
    const size_t esz = dt == TPPO_BF16 ? 2 : 4;
    return tiled_workspace(M) + ((size_t)H * esz % 16 != 0 ? packed_bytes(M, H, V, esz) : 0);
}

extern "C" int tppo_token_logprobs(const void* hidden, int64_t n_rows, int64_t H, int64_t ld_hidden,
                                   const void* w_head, int64_t V, int64_t ld_w, tppo_dtype dt,
                                   const int32_t* sel_rows, const int32_t* sel_targets, int64_t M,
                                   const int64_t* m_actual, const int32_t* out_index, float* logp,
                                   float* lse, void* workspace, size_t workspace_bytes,
                                   int32_t* status, void* stream) {
    using namespace tppo;
    if (dt != TPPO_F32 && dt != TPPO_BF16) return TPPO_ERR_DTYPE;
    if (M < 0 || H < 0 || V < 0 || n_rows < 0 || M > INT32_MAX || V > INT32_MAX - 4096 ||
        H > INT32_MAX)
        return TPPO_ERR_SIZE;
    if (M == 0) return TPPO_OK;
    if (H == 0 || V == 0 || n_rows == 0 || ld_hidden < H || ld_w < H) return TPPO_ERR_SIZE;
    if (!hidden || !w_head || !sel_rows || !sel_targets || !logp) return TPPO_ERR_NULL;
    hipStream_t s = static_cast<hipStream_t>(stream);

    const size_t esz = dt == TPPO_BF16 ? 2 : 4;
    const bool bf16 = dt == TPPO_BF16, have_ws = workspace && is_aligned(workspace, 256);
    // Copies are needed of an operand whose rows are not addressable -- and of both when H itself is ragged, since
    // the sweep runs over the padded H then.
    const bool ragged = (size_t)H * esz % 16 != 0;
    const bool pack_h = ragged || !rows_addressable(hidden, ld_hidden, H, esz);
    const bool pack_w = ragged || !rows_addressable(w_head, ld_w, H, esz);
    const size_t tiled = tiled_workspace(M), copies = packed_bytes(pack_h ? M : 0, H, pack_w ? V : 0, esz);
    // bf16 rows of whole stages at aligned addresses: such a call needs its workspace and the whole chip; any
    // other one has the generic kernel to fall back on, and its limit on H
    const bool matrix_only = bf16 && !pack_h && !pack_w && H % 64 == 0;
    if (!matrix_only && H > kGenMaxH) return TPPO_ERR_SIZE;
    bool fits = have_ws && workspace_bytes >= tiled + ((pack_h || pack_w) ? copies : 0);
    if (matrix_only && !fits) return TPPO_ERR_WORKSPACE;
    if (!matrix_only) fits = fits && device_compute_units() == kSweepGroups;
    if (!fits) {
        return bf16 ? head_generic<uint16_t>(hidden, n_rows, H, ld_hidden, w_head, V, ld_w, sel_rows, sel_targets, M,
                                             m_actual, out_index, logp, lse, status, s)
                    : head_generic<float>(hidden, n_rows, H, ld_hidden, w_head, V, ld_w, sel_rows, sel_targets, M,
                                          m_actual, out_index, logp, lse, status, s);
    }
    HeadParams p = {};
    p.hidden = hidden;
    p.w = w_head;
    p.sel_rows = sel_rows;
    p.sel_targets = sel_targets;
    p.m_actual = m_actual;
    p.n_rows = n_rows; p.ld_h = ld_hidden; p.ld_w = ld_w;
    p.H = (int)H;
    return bf16 ? head_call<uint16_t>(p, M, V, out_index, logp, lse, workspace, tiled, pack_h, pack_w, matrix_only, status, s)
                : head_call<float>(p, M, V, out_index, logp, lse, workspace, tiled, pack_h, pack_w, matrix_only, status, s);
}

extern "C" int tppo_version(void) { return TPPO_VERSION; }
