// tppo_ppo_losses: clipped surrogate (Eq. (ppoloss)) and clipped value loss
// (Eqs. (valueclip), (valueloss)) as masked streaming reductions over the
// response-packed arrays.  Token sets follow Sec. 3.2: policy tokens are the
// first keep_len[i] window tokens of each sequence, value tokens all window
// tokens of finished sequences.  No token depends on another, so the pass walks
// the arrays in aligned frames of 1024 tokens (plan.h), four consecutive tokens
// per thread: a frame's descriptor names the sequence of its first token, and
// a thread whose four tokens lie inside that sequence (all threads of most
// frames) knows its share of both sets from two comparisons.  Of a frame of more than
// two sequences the workgroup fetches the others' metadata into LDS (but for batches of
// windows of a few tokens, loss_fetches).
// No mask array is read, and a thread with no member of a set issues no loads
// for that set (but for what is asked for before the plan is known: all arrays in
// grids of few workgroups, the first frame's policy arrays in others of the
// pass that writes derivatives, loss_load_ahead).
//
// One launch per call.  A persistent grid walks the frames; a thread issues all loads of its share of a
// frame at once (non-temporal 16-byte accesses, consecutive lanes on consecutive 16 bytes, no branch and no wait
// between them), and the many co-resident wavefronts cover each other's memory latency: there is deliberately
// no software pipeline, whose second register set would halve the wavefronts per CU while the compiler, unable
// to count loads issued under a predicate, waits for all of them anyway.  Sums are token-level (Sec. 4.1.1): a
// term is fp32, every sum of terms fp64, in a fixed order, no float atomics -> bit-identical reruns.
// Each workgroup publishes its partial sums as tagged words (plan.h); the
// workgroup with the highest id -- dispatched last -- waits for all of them
// (bounded), adds them up in a fixed order and writes the result, which saves
// the second launch a separate finalisation kernel would cost.
#include <stdlib.h>

#include "plan.h"

namespace tppo {

#ifndef TPPO_LOSS_THREADS
#define TPPO_LOSS_THREADS 256
#endif
constexpr int kLossThreads = TPPO_LOSS_THREADS;
constexpr int kLossParts = kTileTokens / (4 * kLossThreads);      // a workgroup takes this fraction of a frame, four tokens per thread
static_assert(kLossParts >= 1 && kLossParts * 4 * kLossThreads == kTileTokens, "whole parts of a frame");
// Most workgroups of the persistent grids.  Enough of them to keep the memory busy, and no more: the one that collects
// the sums reads 4 (forward) or 8 words of each.  Measured, us, 2048 / 1024 / 768 / 512 workgroups: forward 10.3 / 10.1 / 9.9 /
// 10.8 on 2.3 M tokens in 512 sequences, 14.3 / 15.6 / 17.4 / 21.2 on 3.0 M in 6008, 31.8 / 31.5 / 31.0 / 31.4 on 10 M in 2200, 59.7 / 59.0 /
// 57.0 / 57.7 on 20 M in 4400; with derivatives 16.0 / 15.7 / 15.0 / 16.8, 20.7 / 20.1 / 22.8 / 27.4, 49.5 / 49.1 / 48.3 / 53.3 and 98.0 / 93.1 / 91.5 /
// 102.5: short windows want many.
constexpr int kLossGroups = 1024, kGradGroups = 1024;
constexpr int kFinishSpin = 1 << 20;
// Grids of up to so many workgroups, a frame each, are bound by their round trips: what they may need is asked for at once
// (loss_load_ahead).  us, at most 256 -> 512 -> 1024 of them: 324 K tokens losses 6.26 -> 5.80 -> 5.83, derivatives 8.04 -> 7.66 -> 7.63;
// 571 K 6.80 -> 6.8 -> 7.06, 9.53 -> 9.5 -> 9.10;  872 K 7.6 -> 7.6 -> 7.2, 10.1 -> 10.1 -> 10.3;  878 K, a tenth of the sequences finished,
// 7.1 -> 7.1 -> 7.1, 9.4 -> 9.4 -> 9.6: beyond 512 what is asked for in vain costs as much as the trips.
constexpr int kFewGroups = 512;
static_assert(kFewGroups <= kLossGroups && kFewGroups <= kGradGroups, "a frame to a workgroup");

struct LossParams {
    const float *logp_new, *logp_old, *adv, *v_new, *v_old, *ret;
    const int32_t *resp_off, *keep_len, *done;
    void* plan;
    int32_t* status;
    int B, n_resp;
    uint32_t tag;
    float ratio_lo, ratio_hi, xi_low, xi_high;
    int all_ahead;                     // loss_load_ahead
};

typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));   // 16-byte access, 4-byte aligned

// exp for the probability ratio: one multiply and the hardware exp2 (relative error ~1e-7 (1 + |x|), far inside
// the tolerances; the library expf costs ~15 more instructions per token)
__device__ __forceinline__ float ratio_exp(float x) {
    return __builtin_amdgcn_exp2f(x * 1.4426950408889634f);
}

__device__ __forceinline__ float clampf(float x, float lo, float hi) {
    return fminf(fmaxf(x, lo), hi);
}

// fminf / fmaxf return the operand that IS a number, so a NaN input would be clipped away; inside a token set
// it must reach the result instead (the term of such a token is undefined), hence the explicit tests.
__device__ __forceinline__ float surrogate(float ln, float lo, float a, float rlo, float rhi) {
    const float rho = ratio_exp(ln - lo);
    const float u = rho * a;
    const float t = fminf(u, clampf(rho, rlo, rhi) * a);
    return u != u ? u : t;
}

__device__ __forceinline__ bool value_undefined(float d0, float d1, float vo) {
    return d0 != d0 || d1 != d1 || vo != vo;
}

__device__ __forceinline__ float value_term(float v, float vo, float r, float xl, float xh) {
    const float d0 = v - r;
    const float d1 = clampf(v, vo - xl, vo + xh) - r;
    return value_undefined(d0, d1, vo) ? __builtin_nanf("") : fmaxf(d0 * d0, d1 * d1);
}

// The workgroup's sums of kSums values per thread, in a fixed order: a wavefront's by data-parallel moves, its last lane leaves them in
// LDS, and after the one barrier whoever needs a sum adds up the wavefronts' with block_sum.  (Through shuffles, two barriers and a
// loop over the launch's wavefront count, read from memory, a small batch took 0.7 to 2 us for two sums and 1.4 to 2.7 for five.)
// s_red: kSums * (wavefronts of the workgroup) doubles.
template <int kSums>
__device__ __forceinline__ void block_sums(const double (&x)[kSums], double* s_red) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < kSums; ++q) {
        const double t = wave_prefix(x[q]);
        if (lane == kWave - 1) s_red[wave * kSums + q] = t;
    }
    __syncthreads();
}
template <int kSums, int kWaves>
__device__ __forceinline__ double block_sum(const double* s_red, int q) {
    double t = s_red[q];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) t += s_red[w * kSums + q];
    return t;
}

// Four consecutive results per access; `n` = how many of the four exist.
__device__ __forceinline__ void store4(float* __restrict__ dst, int first, const float (&x)[4], int n) {
    if (n >= 4) {
        float4u t;
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = x[e];
        __builtin_nontemporal_store(t, reinterpret_cast<float4u*>(dst + first));
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (e < n) dst[first + e] = x[e];
    }
}

// What one thread holds of one frame: 16 bytes of each of the six arrays.
struct LossRegs {
    float4u ln, lo, a, v, vo, r;
};

// A thread's four consecutive tokens: the first one's index, how many of the four exist, and which are policy /
// value tokens (bit e: token first + e).
struct TokenSets {
    int first, n_tok, pol, val;
};

// The metadata of the sequences that follow the two a frame's descriptor knows, one per thread of the workgroup: one round
// trip.  Every thread behind the second boundary looking for itself, token by token and from the fourth sequence on by
// bisection in memory, took, us: 3.0 M tokens in 6008 sequences losses 23.0 (now 16.1), derivatives 31.9 (23.7);  3.4 M in
// 2703: 18.9 (16.3), 28.0 (23.6);  8.2 M in 3260: 32.2 (27.8), 47.1 (44.4).  A sequence's
// four words are one read of LDS: as four arrays, read token by token, 19.0 and 26.5 at 3.0 M.  (All of these, and those below, with sums
// through shuffles, on both sides; a pass of the first takes 15.4 now.)
// The policy arrays wait for the lookup, but for those that loss_load_ahead asks for: short unfinished sequences keep few tokens or
// none.  Asked for by every thread beside the metadata instead, with 0.2 / 0.5 / 0.8 / 1 of 3.0 M tokens in windows of 64 .. 512 kept: losses 15.9 / 16.8 / 17.1 / 17.0 (now
// 14.9 / 16.0 / 16.7 / 17.4), derivatives 23.9 / 25.2 / 25.6 / 26.0 (22.7 / 23.7 / 24.1 / 24.9); the three layouts above 16.0, 16.2,
// 28.1 and 24.2, 24.1, 44.7.  (Grids of few workgroups, which wait for nothing else, are faster so: kFewGroups.)
struct MoreSeqs {
    int4 seq[kLossThreads];                      // a sequence's first token, its end, the end of its policy tokens, finished
    int in_frame[kLossThreads / kWave];          // how many of a wavefront's begin before the frame's end
};
struct SeqMeta {
    int lo, hi, keep, fin;
};
__host__ __device__ __forceinline__ SeqMeta load_meta(const LossParams& p, int i) {
    const int at = min(i, p.B - 1);
    return SeqMeta{p.resp_off[at], p.resp_off[at + 1], p.keep_len[at], p.done[at]};
}
__host__ __device__ __forceinline__ int4 kept_words(const SeqMeta& x) {
    return make_int4(x.lo, x.hi, x.lo + min(max(x.keep, 0), x.hi - x.lo), x.fin);
}
// (`more`: another one than the last time, which other threads may still look at)
__device__ __forceinline__ void keep_meta(MoreSeqs& more, const SeqMeta& x, bool exists, int frame_end, int tid) {
    const uint64_t in_frame = __ballot(exists && x.lo < frame_end);
    if ((tid & 63) == 0) more.in_frame[tid >> 6] = __popcll(in_frame);
    more.seq[tid] = kept_words(x);
    __syncthreads();
}

// The sets of the tokens at or beyond `end` of sequence `seg` (the last one that is known without a look into memory):
// token by token, moving on to the sequence that holds the token -- normally the next one, whose four
// metadata words are asked for together; past empty sequences by bisection of the offsets, so the work is
// bounded whatever the layout.  Offsets that are not a layout (decreasing, beyond the arrays) put a token in
// no set; they cannot make an access leave the arrays.
__host__ __device__ __forceinline__ void walk_sets(const LossParams& p, int seg, int end, TokenSets& ts) {
    int pol_end = end;
    bool fin = false, inside = false;
    for (int e = 0; e < ts.n_tok; ++e) {
        const int q = ts.first + e;
        if (q < end && !inside) continue;                          // a token the descriptor covered
        if (q >= end) {                                            // find the sequence that holds q
            int nxt = seg + 1;
            if (nxt >= p.B) break;                                 // beyond the last sequence
            int lo = p.resp_off[nxt], hi = p.resp_off[nxt + 1], keep = p.keep_len[nxt], dn = p.done[nxt];
            if (hi <= q) {                                         // not the next one: the last sequence that begins at or before q
                int a = nxt + 1, b = p.B - 1;
                if (a > b) break;
                while (a < b) {
                    const int m = (a + b + 1) >> 1;
                    if (p.resp_off[m] <= q) a = m; else b = m - 1;
                }
                nxt = a;
                lo = p.resp_off[nxt]; hi = p.resp_off[nxt + 1]; keep = p.keep_len[nxt]; dn = p.done[nxt];
            }
            inside = q >= lo && q < hi;
            if (!inside) continue;                                 // no sequence holds q (seg, end unchanged: look again)
            seg = nxt;
            end = hi;
            pol_end = lo + min(max(keep, 0), hi - lo);
            fin = dn != 0;
        }
        ts.pol |= q < pol_end ? 1 << e : 0;
        ts.val |= fin ? 1 << e : 0;
    }
}

// The same, looked up in what the workgroup has fetched of the sequences behind `seg`, of which the first `past` end at or before `end`:
// the first one that ends beyond a thread's first token by bisection, the others from there on.  Only tokens beyond all of them walk on.
__host__ __device__ __forceinline__ void more_sets(const LossParams& p, const MoreSeqs& more, int seg, int past, int end, TokenSets& ts) {
    int count = 0;
#pragma unroll
    for (int w = 0; w < kLossThreads / kWave; ++w) count += more.in_frame[w];
    const int from = max(ts.first, end);
    int j = min(past, count), above = count;
    while (j < above) {
        const int m = j + ((above - j) >> 1);
        if (more.seq[m].y <= from) j = m + 1; else above = m;
    }
    int4 x = more.seq[min(j, kLossThreads - 1)];
    for (int e = 0; e < ts.n_tok; ++e) {
        const int q = ts.first + e;
        if (q < end) continue;                                     // a token the descriptor covered
        while (j < count && x.y <= q) {
            ++j;
            x = more.seq[min(j, kLossThreads - 1)];
        }
        if (j == count) {
            if (count == kLossThreads && seg + count < p.B - 1) walk_sets(p, seg + count, x.y, ts);
            break;
        }
        if (q < x.x) continue;                                     // no sequence holds q
        ts.pol |= q < x.z ? 1 << e : 0;
        ts.val |= x.w != 0 ? 1 << e : 0;
    }
}

// A frame with tokens behind the two sequences its descriptor knows: the same for the whole workgroup, which has `seqs` filled
// then and only then.
__host__ __device__ __forceinline__ bool has_more(const LossParams& p, const FrameDesc& d, int item) {
    return d.end2 < min((item + 1) * (4 * kLossThreads), p.n_resp) && d.seg2 + 1 < p.B;
}

// from: the first sequence that was fetched (< 0: the one after the two that the descriptor knows)
template <bool kFetch>
__host__ __device__ __forceinline__ TokenSets token_sets(const LossParams& p, const FrameDesc& d, bool more, const MoreSeqs& seqs,
                                                         int item, int tid, bool has_pol, bool has_val, int from = -1) {
    TokenSets ts;
    ts.first = item * (4 * kLossThreads) + 4 * tid;                // item: part item % kLossParts of frame item / kLossParts
    ts.n_tok = min(max(p.n_resp - ts.first, 0), 4);
    if (ts.first + 4 <= d.end) {                                   // all four in the frame's first sequence
        ts.pol = (1 << min(max(d.pol_end - ts.first, 0), 4)) - 1;
        ts.val = d.fin != 0 ? 0xF : 0;
    } else {                                                       // token by token: first sequence, second, or beyond
        ts.pol = ts.val = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int q = ts.first + e;
            const bool in1 = q < d.end, in2 = !in1 && q < d.end2;
            ts.pol |= ((in1 && q < d.pol_end) || (in2 && q < d.pol_end2)) ? 1 << e : 0;
            ts.val |= ((in1 && d.fin != 0) || (in2 && d.fin2 != 0)) ? 1 << e : 0;
        }
        // (a thread beyond the end of the arrays has no token to look for)
        if ((more || !kFetch) && ts.n_tok > 0 && ts.first + ts.n_tok > d.end2) {
            if (kFetch) more_sets(p, seqs, from < 0 ? d.seg2 : from - 1, from < 0 ? 0 : d.seg2 + 1 - from, d.end2, ts);
            else walk_sets(p, d.seg2, d.end2, ts);
        }
    }
    ts.pol = (has_pol && ts.n_tok > 0) ? ts.pol & ((1 << ts.n_tok) - 1) : 0;
    ts.val = (has_val && ts.n_tok > 0) ? ts.val & ((1 << ts.n_tok) - 1) : 0;
    return ts;
}

// A frame's descriptor, checked: a plan is caller-held memory.  Whatever it says, no access leaves the arrays
// (tokens are addressed by frame and thread, not through the descriptor); only `seg2` indexes the metadata.
__device__ __forceinline__ FrameDesc checked_frame(FrameDesc d, const LossParams& p, int tid) {
    if (d.seg < 0 || d.seg >= p.B || d.seg2 < 0 || d.seg2 >= p.B) {
        if (tid == 0) set_status(p.status, TPPO_STATUS_BAD_LAYOUT);
        d = FrameDesc{p.B - 1, 0, 0, 0, p.B - 1, 0, 0, 0};         // every token looks for its sequence itself and finds none
    }
    return d;
}

// Issue the loads of a thread's four tokens, one set's arrays each.  Consecutive lanes on consecutive 16 bytes (the access shape that
// streams at full rate), non-temporal.  Nothing is loaded for a set none of the four is in; with 1..3 members
// the 16 bytes are loaded whole -- the surplus elements are never used -- so that no branch and no wait
// separates the loads and all of them are in flight together; the one thread that would read past the END OF
// THE ARRAY reads the array's last 16 bytes instead (see unshift).  Needs n_resp >= 4.
__device__ __forceinline__ void loss_load_policy(LossRegs& x, const LossParams& p, const TokenSets& ts) {
    const int at = min(ts.first, p.n_resp - 4);
    if (ts.pol != 0) {
        x.ln = __builtin_nontemporal_load(reinterpret_cast<const float4u*>(p.logp_new + at));
        x.lo = __builtin_nontemporal_load(reinterpret_cast<const float4u*>(p.logp_old + at));
        x.a = __builtin_nontemporal_load(reinterpret_cast<const float4u*>(p.adv + at));
    }
}
__device__ __forceinline__ void loss_load_value(LossRegs& x, const LossParams& p, const TokenSets& ts) {
    const int at = min(ts.first, p.n_resp - 4);
    if (ts.val != 0) {
        x.v = __builtin_nontemporal_load(reinterpret_cast<const float4u*>(p.v_new + at));
        x.vo = __builtin_nontemporal_load(reinterpret_cast<const float4u*>(p.v_old + at));
        x.r = __builtin_nontemporal_load(reinterpret_cast<const float4u*>(p.ret + at));
    }
}

// What a workgroup asks for before the plan is known, so that the plan's header, the frame's descriptor and these are one round trip
// instead of three:
//   the first frame's policy arrays, in the pass that writes derivatives: all but the dropped tails are policy tokens, so little
//     of it is asked for in vain.  Derivatives alone, us, after the descriptor -> so, at a tenth / three tenths / nine tenths of finished
//     sequences: 1 M tokens 16.6 / 17.3 / 18.0 -> 15.7 / 16.8 / 17.4;  4 M 25.8 / 27.2 / 31.0 -> 25.7 / 26.7 / 30.8 (with sums through
//     shuffles, on both sides).
//   kFew, a grid of so few workgroups (kFewGroups) that latency is all they take: all six arrays, and all sequences' metadata, one per
//     thread, if there are no more (all_ahead), for frames with more sequences than the two that the descriptor knows.
template <bool kFew>
__device__ __forceinline__ void loss_load_ahead(LossRegs& x, SeqMeta& all, const LossParams& p, int tid) {
    const int at = min((int)blockIdx.x * (4 * kLossThreads) + 4 * tid, p.n_resp - 4);
    if (p.logp_new) {
        x.ln = __builtin_nontemporal_load(reinterpret_cast<const float4u*>(p.logp_new + at));
        x.lo = __builtin_nontemporal_load(reinterpret_cast<const float4u*>(p.logp_old + at));
        x.a = __builtin_nontemporal_load(reinterpret_cast<const float4u*>(p.adv + at));
    }
    if (kFew && p.v_new) {
        x.v = __builtin_nontemporal_load(reinterpret_cast<const float4u*>(p.v_new + at));
        x.vo = __builtin_nontemporal_load(reinterpret_cast<const float4u*>(p.v_old + at));
        x.r = __builtin_nontemporal_load(reinterpret_cast<const float4u*>(p.ret + at));
    }
    if (kFew && p.all_ahead) all = load_meta(p, tid);
}

// kFew: by one and by two places, a few selects, where the end of the array is somebody's last frame and everybody waits for it (us, one select
// of four for each -> so: 126 tokens losses 5.0 -> 4.2, derivatives 6.2 -> 5.4;  49 K 6.2 -> 5.5, 7.8 -> 7.1).  The loops over many frames
// are scheduled worse around it (40 M tokens, derivatives 165 -> 169) and keep the other.
template <bool kFew>
__device__ __forceinline__ float4u rotate_left(float4u t, int sh) {
    float4u o;
    if constexpr (kFew) {
        float4u by1;
#pragma unroll
        for (int e = 0; e < 4; ++e) by1[e] = sh & 1 ? t[(e + 1) & 3] : t[e];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = sh & 2 ? by1[(e + 2) & 3] : by1[e];
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            o[e] = sh == 0 ? t[e] : sh == 1 ? t[(e + 1) & 3] : sh == 2 ? t[(e + 2) & 3] : t[(e + 3) & 3];
    }
    return o;
}

// the array's last few tokens were loaded as part of its last 16 bytes: move them into place (only in the last
// frame, and there for at most one thread)
template <bool kFew>
__device__ __forceinline__ void unshift(LossRegs& x, const TokenSets& ts, int item, int n_resp) {
    if (__builtin_expect((item + 1) * (4 * kLossThreads) <= n_resp, 1)) return;   // wave-uniform: not the array's end
    if (kFew && (n_resp & 3) == 0) return;                                        // ... or four by four up to it
    const int sh = ts.n_tok > 0 ? max(ts.first - (n_resp - 4), 0) : 0;
    x.ln = rotate_left<kFew>(x.ln, sh); x.lo = rotate_left<kFew>(x.lo, sh); x.a = rotate_left<kFew>(x.a, sh);
    x.v = rotate_left<kFew>(x.v, sh); x.vo = rotate_left<kFew>(x.vo, sh); x.r = rotate_left<kFew>(x.r, sh);
}

// A workgroup publishes kWords words: of each of kSums - kCounts sums two (a double as hi + lo), of each of the kCounts last ones, whole
// numbers up to 2^24 (countable), one.
template <int kSums, int kCounts>
struct SumWords {
    static constexpr int kFloats = 2 * (kSums - kCounts), kWords = kFloats + kCounts;
    static_assert(kWords <= kFinishWords && kLossThreads % kWords == 0, "a workgroup's words, and threads that read one kind of them only");
    __device__ static __forceinline__ void publish_sum(unsigned long long* mine, uint32_t tag, int q, double x) {
        if (q < kSums - kCounts) publish(mine + 2 * q, tag, x);
        else __hip_atomic_store(mine + kFloats + q - (kSums - kCounts), pack_word(tag, (float)x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
};

// The sums of all workgroups, collected by the one with the highest id: valid in the last lane of its first wavefront.  The words lie one
// after the other; consecutive threads read consecutive ones, every thread words of one kind only, kBatch of them asked for
// together (bypassing the caches: each a trip to memory; with a thread to a workgroup's words, 80 bytes apart, the
// requests were ten times as many), and again, bounded, until all of them are there.  Every thread adds up its words in order,
// then the threads of a kind are added up in a fixed tree: deterministic.  False in *s_flag when a wait gave up.
template <int kSums, int kCounts>
__device__ __forceinline__ void collect_sums(const unsigned long long* words, uint32_t tag, int groups, double (&tot)[kSums],
                                             double* s_fin, int* s_flag) {
    typedef SumWords<kSums, kCounts> Words;
    constexpr int kWords = Words::kWords, kPart = kLossThreads / kWords, kBatch = 16;
    static_assert(kFinishGroups * kFinishWords % (kLossThreads * kBatch) == 0, "whole batches stay within the plan's words");
    const unsigned tid = threadIdx.x, lane = tid & 63;
    const int n = groups * kWords;
    double acc = 0.0;
    bool ok = true;
    for (int first = 0; first < n; first += kLossThreads * kBatch) {
        const int left = n - first - (int)tid;                     // of mine from here on: b * kLossThreads < left
        unsigned long long w[kBatch];
        uint32_t missing = 1;
        for (int spin = 0; spin < kFinishSpin && missing != 0; ++spin) {
            if (spin > 0) __builtin_amdgcn_s_sleep(1);
            unsigned at = tid;
            asm volatile("" : "+v"(at));                           // (no address kept over the rounds: the registers are full)
            missing = 0;
#pragma unroll
            for (int b = 0; b < kBatch; ++b)
                if (b * kLossThreads < n - first)
                    w[b] = __hip_atomic_load(words + first + b * kLossThreads + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int b = 0; b < kBatch; ++b) missing |= b * kLossThreads < left ? (uint32_t)(w[b] >> 32) ^ tag : 0;
        }
        ok = ok && missing == 0;
#pragma unroll
        for (int b = 0; b < kBatch; ++b) acc += b * kLossThreads < left ? (double)__uint_as_float((unsigned)w[b]) : 0.0;
    }
    s_fin[tid] = acc;
    if (!ok) *s_flag = 0;
    __syncthreads();
    if (tid >= kWave) return;
#pragma unroll
    for (int q = 0; q < kSums; ++q) {
        double t = 0.0;
        for (unsigned k = lane; k < kPart; k += kWave) {
            const double* of = s_fin + k * kWords;
            t += q < kSums - kCounts ? of[2 * q] + of[2 * q + 1] : of[q + kSums - kCounts];
        }
        tot[q] = wave_prefix(t);
    }
}

// A workgroup's sums (block_sums) become the batch's, in the last lane of a wavefront for which this returns true: at once in a grid of
// one, else in the workgroup with the highest id, all others having published theirs.  s_flag was set before block_sums.
template <int kSums, int kCounts>
__device__ __forceinline__ bool finish_sums(unsigned long long* words, uint32_t tag, double (&tot)[kSums],
                                            const double* s_red, double* s_fin, int* s_flag) {
    constexpr int kWaves = kLossThreads / kWave;
    const int tid = threadIdx.x;
    if (gridDim.x == 1) {
#pragma unroll
        for (int q = 0; q < kSums; ++q) tot[q] = block_sum<kSums, kWaves>(s_red, q);
        return tid == kWave - 1;
    }
    typedef SumWords<kSums, kCounts> Words;
    if (tid < kSums) Words::publish_sum(words + blockIdx.x * Words::kWords, tag, tid, block_sum<kSums, kWaves>(s_red, tid));
    if (blockIdx.x != gridDim.x - 1) return false;
    collect_sums<kSums, kCounts>(words, tag, (int)gridDim.x, tot, s_fin, s_flag);
    return tid == kWave - 1;
}

__device__ __forceinline__ void write_losses(tppo_loss_out* out, double pol_terms, double val_terms, long long np,
                                             long long nv) {
    const double policy_sum = -pol_terms, value_sum = 0.5 * val_terms;   // policy_loss = -J_PPO
    out->policy_sum = (float)policy_sum;
    out->value_sum = (float)value_sum;
    out->policy_loss = np > 0 ? (float)(policy_sum / (double)np) : 0.f;
    out->value_loss = nv > 0 ? (float)(value_sum / (double)nv) : 0.f;
    out->n_policy = np;
    out->n_value = nv;
}

// what a call that could not compute leaves behind: not a number, so that nobody trains on it
__device__ __forceinline__ void write_invalid(tppo_loss_out* out) {
    out->policy_sum = out->value_sum = out->policy_loss = out->value_loss = __builtin_nanf("");
    out->n_policy = out->n_value = 0;
}

// (The lookup's scalar registers leave seven wavefronts a SIMD.  Held to eight, which spills them, us, seven -> eight: 129 tokens 4.2 ->
// 4.5, 4521 in 100 sequences 5.7 -> 6.2, 43 K in 100 5.3 -> 5.6, 2.3 M in 512 9.6 -> 9.9, 3.0 M in 6008 15.4 -> 16.3, 20 M 58.7 -> 59.2.)
template <bool kFetch, bool kFew>
__global__ __launch_bounds__(kLossThreads, kFetch ? 6 : 8) void loss_kernel(LossParams p, tppo_loss_out* __restrict__ out) {
    __shared__ double s_red[2 * kLossThreads / kWave], s_fin[kLossThreads];
    __shared__ int s_flag;
    __shared__ MoreSeqs s_more[2];
    const int tid = threadIdx.x;
    LossRegs first = {};
    SeqMeta all = {};
    if (kFew) loss_load_ahead<kFew>(first, all, p, tid);
    const Plan pl = plan_open(p.plan);
    const bool has_pol = p.logp_new != nullptr, has_val = p.v_new != nullptr;
    const bool plan_ok = pl.hdr->B == p.B && pl.hdr->n_resp == p.n_resp && pl.hdr->has_sets != 0 &&
                         pl.cap >= p.n_resp / kTileTokens + p.B + 1;
    if (!plan_ok) {                                                // not this batch's plan: touch nothing of it
        if (blockIdx.x == 0 && tid == 0) {
            set_status(p.status, TPPO_STATUS_BAD_LAYOUT);
            write_invalid(out);
        }
        return;
    }
    const int count = (p.n_resp + 4 * kLossThreads - 1) / (4 * kLossThreads);     // work items: parts of frames

    double pol_acc = 0.0, val_acc = 0.0;
    FrameDesc ahead = {};
    int which = 0;                                                 // of s_more
    if ((int)blockIdx.x < count) ahead = load_frame(pl.frames + blockIdx.x / kLossParts);
    for (int f = blockIdx.x; f < count; f += gridDim.x) {
        const FrameDesc d = checked_frame(ahead, p, tid);
        if (f + (int)gridDim.x < count) ahead = load_frame(pl.frames + (f + gridDim.x) / kLossParts);     // the next item's, meanwhile
        const bool more = kFetch && has_more(p, d, f);
        const int from = kFew && p.all_ahead ? 0 : d.seg2 + 1;
        if (more) {
            const SeqMeta meta = kFew && p.all_ahead ? all : load_meta(p, from + tid);
            which ^= 1;
            keep_meta(s_more[which], meta, from + tid < p.B, (f + 1) * (4 * kLossThreads), tid);
        }
        const TokenSets ts = token_sets<kFetch>(p, d, more, s_more[which], f, tid, has_pol, has_val, from);
        LossRegs cur = first;
        if (!kFew) {
            loss_load_policy(cur, p, ts);
            loss_load_value(cur, p, ts);
        }
        unshift<kFew>(cur, ts, f, p.n_resp);
        float pol_t = 0.f, val_t = 0.f;                            // this thread's <= 8 terms of the frame
        if (ts.pol != 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float t = surrogate(cur.ln[e], cur.lo[e], cur.a[e], p.ratio_lo, p.ratio_hi);
                pol_t += (ts.pol >> e & 1) ? t : 0.f;              // select, never multiply by a mask
            }
        }
        if (ts.val != 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float t = value_term(cur.v[e], cur.vo[e], cur.r[e], p.xi_low, p.xi_high);
                val_t += (ts.val >> e & 1) ? t : 0.f;
            }
        }
        pol_acc += (double)pol_t;
        val_acc += (double)val_t;
        if (kFew) break;                                           // (a frame to a workgroup)
    }
    double tot[2] = {pol_acc, val_acc};
    if (tid == 0) s_flag = 1;
    block_sums(tot, s_red);
    if (finish_sums<2, 0>(pl.finish_words, p.tag, tot, s_red, s_fin, &s_flag)) {
        if (s_flag == 0) {
            set_status(p.status, TPPO_STATUS_TIMEOUT);
            tot[0] = tot[1] = __builtin_nan("");
        }
        write_losses(out, tot[0], tot[1], has_pol ? pl.hdr->n_policy : 0,
                     has_val ? pl.hdr->n_value : 0);
    }
}

// nothing to sum (no tokens, or neither half asked for): both sets are empty
__global__ void loss_empty_kernel(tppo_loss_out* __restrict__ out, tppo_loss_stats* __restrict__ stats) {
    if (threadIdx.x != 0) return;
    if (out) write_losses(out, 0.0, 0.0, 0, 0);
    if (stats) {
        stats->ratio_mean = stats->policy_clip_frac = stats->value_clip_frac = stats->reserved = 0.f;
        stats->n_policy_clipped = stats->n_value_clipped = 0;
    }
}

// ---------------------------------------------------------------------------
// tppo_ppo_losses_backward: the same streaming pass, also writing the
// derivatives of the two losses with respect to logp_new and v_new and
// counting the tokens whose clip is active.
//   policy token: surrogate min(u, c), u = rho A, c = clip(rho) A.  Where
//     u <= c the unclipped branch is the minimum (inside the clip range both
//     are the same function) and d/dlogp_new = rho A; where c < u the clip is
//     saturated, c is constant, the derivative is 0.
//   value token: 1/2 max(d0^2, d1^2), d0 = V - R, d1 = V_clip - R.  Where
//     d0^2 >= d1^2 the derivative is d0; otherwise V is outside the clip
//     range, V_clip is constant and the derivative is 0.
//   a token with a NaN among its inputs: the derivative is NaN, and it counts
//     neither as clipped nor as unclipped.
// Token-level means: the set sizes are known from the metadata before the pass
// (the plan holds them), so each derivative is final when it is written; tokens
// outside a set get 0.
constexpr int kGradSums = 5;       // policy terms, value terms, ratios, clipped policy tokens, clipped value tokens

struct GradParams {
    LossParams fwd;
    float* grad_logp;
    float* grad_v;
    float policy_scale, value_scale;
    long long policy_denominator, value_denominator;     // <= 0: the call's own token counts
};

template <bool kFetch, bool kFew>
__global__ __launch_bounds__(kLossThreads, 4) void loss_grad_kernel(GradParams gp, tppo_loss_out* __restrict__ out,
                                                                    tppo_loss_stats* __restrict__ stats) {
    __shared__ double s_red[kGradSums * kLossThreads / kWave], s_fin[kLossThreads];
    __shared__ int s_flag;
    __shared__ MoreSeqs s_more[2];
    const LossParams& p = gp.fwd;
    const int tid = threadIdx.x;
    LossRegs cur = {};
    SeqMeta all = {};
    loss_load_ahead<kFew>(cur, all, p, tid);
    const Plan pl = plan_open(p.plan);
    const bool has_pol = p.logp_new != nullptr, has_val = p.v_new != nullptr;
    const bool plan_ok = pl.hdr->B == p.B && pl.hdr->n_resp == p.n_resp && pl.hdr->has_sets != 0 &&
                         pl.cap >= p.n_resp / kTileTokens + p.B + 1;
    if (!plan_ok) {                                                // not this batch's plan: touch nothing of it
        if (blockIdx.x == 0 && tid == 0) {
            set_status(p.status, TPPO_STATUS_BAD_LAYOUT);
            if (out) write_invalid(out);
        }
        return;
    }
    const int count = (p.n_resp + 4 * kLossThreads - 1) / (4 * kLossThreads);     // work items: parts of frames
    const long long np = has_pol ? pl.hdr->n_policy : 0, nv = has_val ? pl.hdr->n_value : 0;
    const long long den_p = gp.policy_denominator > 0 ? gp.policy_denominator : np;
    const long long den_v = gp.value_denominator > 0 ? gp.value_denominator : nv;
    const float pol_coef = den_p > 0 ? -gp.policy_scale / (float)den_p : 0.f;     // policy_loss = -J_PPO
    const float val_coef = den_v > 0 ? gp.value_scale / (float)den_v : 0.f;

    double pol_acc = 0.0, val_acc = 0.0, ratio_acc = 0.0;
    int pol_clipped = 0, val_clipped = 0;
    FrameDesc ahead = {};
    int which = 0;                                                 // of s_more
    if ((int)blockIdx.x < count) ahead = load_frame(pl.frames + blockIdx.x / kLossParts);
    for (int f = blockIdx.x; f < count; f += gridDim.x) {
        const FrameDesc d = checked_frame(ahead, p, tid);
        if (f + (int)gridDim.x < count) ahead = load_frame(pl.frames + (f + gridDim.x) / kLossParts);     // the next item's, meanwhile
        const bool more = kFetch && has_more(p, d, f);
        const int from = kFew && p.all_ahead ? 0 : d.seg2 + 1;
        if (more) {
            const SeqMeta meta = kFew && p.all_ahead ? all : load_meta(p, from + tid);
            which ^= 1;
            keep_meta(s_more[which], meta, from + tid < p.B, (f + 1) * (4 * kLossThreads), tid);
        }
        const TokenSets ts = token_sets<kFetch>(p, d, more, s_more[which], f, tid, has_pol, has_val, from);
        if (f != (int)blockIdx.x) loss_load_policy(cur, p, ts);
        if (!kFew) loss_load_value(cur, p, ts);
        unshift<kFew>(cur, ts, f, p.n_resp);
        float pol_t = 0.f, val_t = 0.f, ratio_t = 0.f;
        if (has_pol && ts.n_tok > 0) {
            float gl[4] = {0.f, 0.f, 0.f, 0.f};
            if (ts.pol != 0) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float rho = ratio_exp(cur.ln[e] - cur.lo[e]);
                    const float u = rho * cur.a[e];
                    const float c = clampf(rho, p.ratio_lo, p.ratio_hi) * cur.a[e];
                    const bool in_set = (ts.pol >> e & 1) != 0, unclipped = u <= c, undefined = u != u;
                    pol_t += in_set ? (undefined ? u : fminf(u, c)) : 0.f;     // select, never multiply by a mask
                    ratio_t += in_set ? rho : 0.f;
                    pol_clipped += (in_set && !unclipped && !undefined) ? 1 : 0;
                    gl[e] = in_set ? (undefined ? u : unclipped ? pol_coef * u : 0.f) : 0.f;
                }
            }
            store4(gp.grad_logp, ts.first, gl, ts.n_tok);
        }
        if (has_val && ts.n_tok > 0) {
            float gv[4] = {0.f, 0.f, 0.f, 0.f};
            if (ts.val != 0) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float d0 = cur.v[e] - cur.r[e];
                    const float d1 = clampf(cur.v[e], cur.vo[e] - p.xi_low, cur.vo[e] + p.xi_high) - cur.r[e];
                    const float q0 = d0 * d0, q1 = d1 * d1;
                    const bool in_set = (ts.val >> e & 1) != 0, unclipped = q0 >= q1;
                    const bool undefined = value_undefined(d0, d1, cur.vo[e]);
                    const float nan = __builtin_nanf("");
                    val_t += in_set ? (undefined ? nan : fmaxf(q0, q1)) : 0.f;
                    val_clipped += (in_set && !unclipped && !undefined) ? 1 : 0;
                    gv[e] = in_set ? (undefined ? nan : unclipped ? val_coef * d0 : 0.f) : 0.f;
                }
            }
            store4(gp.grad_v, ts.first, gv, ts.n_tok);
        }
        pol_acc += (double)pol_t;
        val_acc += (double)val_t;
        ratio_acc += (double)ratio_t;
        if (kFew) break;                                           // (a frame to a workgroup)
    }
    if (!out && !stats) return;                                    // (nobody asks for the sums)
    double tot[kGradSums] = {pol_acc, val_acc, ratio_acc, (double)pol_clipped, (double)val_clipped};
    if (tid == 0) s_flag = 1;
    block_sums(tot, s_red);
    if (finish_sums<kGradSums, 2>(pl.finish_words, p.tag, tot, s_red, s_fin, &s_flag)) {
        const bool ok = s_flag != 0;
        if (!ok) {
            set_status(p.status, TPPO_STATUS_TIMEOUT);
#pragma unroll
            for (int q = 0; q < kGradSums; ++q) tot[q] = __builtin_nan("");
        }
        if (out) write_losses(out, tot[0], tot[1], np, nv);
        if (stats) {
            stats->ratio_mean = np > 0 ? (float)(tot[2] / (double)np) : 0.f;
            stats->policy_clip_frac = np > 0 ? (float)(tot[3] / (double)np) : 0.f;
            stats->value_clip_frac = nv > 0 ? (float)(tot[4] / (double)nv) : 0.f;
            stats->reserved = 0.f;
            stats->n_policy_clipped = ok ? (long long)tot[3] : -1;
            stats->n_value_clipped = ok ? (long long)tot[4] : -1;
        }
    }
}

// Batches of fewer than four tokens (the streaming kernels' 16-byte accesses need four): one workgroup, one
// thread per sequence, token by token from the definitions.  kGrad also writes the derivatives.
template <bool kGrad>
__global__ __launch_bounds__(256) void loss_tiny_kernel(GradParams gp, const int32_t* __restrict__ resp_off,
                                                        tppo_loss_out* __restrict__ out,
                                                        tppo_loss_stats* __restrict__ stats) {
    constexpr int kWaves = 256 / kWave;
    __shared__ double s_cnt[2 * kWaves], s_red[kGradSums * kWaves];
    const LossParams& p = gp.fwd;
    const bool has_pol = p.logp_new != nullptr, has_val = p.v_new != nullptr;
    const int tid = threadIdx.x;
    double cnt_p = 0.0, cnt_v = 0.0;
    for (int i = tid; i < p.B; i += blockDim.x) {
        const int win = max(min(resp_off[i + 1], p.n_resp) - max(resp_off[i], 0), 0);
        if (has_pol) cnt_p += (double)min(max(p.keep_len[i], 0), win);
        if (has_val && p.done[i] != 0) cnt_v += (double)win;
    }
    const double cnt[2] = {cnt_p, cnt_v};
    block_sums(cnt, s_cnt);
    const long long np = (long long)block_sum<2, kWaves>(s_cnt, 0), nv = (long long)block_sum<2, kWaves>(s_cnt, 1);
    const long long den_p = gp.policy_denominator > 0 ? gp.policy_denominator : np;
    const long long den_v = gp.value_denominator > 0 ? gp.value_denominator : nv;
    const float pol_coef = den_p > 0 ? -gp.policy_scale / (float)den_p : 0.f;
    const float val_coef = den_v > 0 ? gp.value_scale / (float)den_v : 0.f;
    double sums[kGradSums] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (int i = tid; i < p.B; i += blockDim.x) {
        const int lo = max(resp_off[i], 0), hi = min(resp_off[i + 1], p.n_resp);
        const int keep = min(max(p.keep_len[i], 0), max(hi - lo, 0));
        const bool fin = p.done[i] != 0;
        for (int t = lo; t < hi; ++t) {
            if (has_pol) {
                float g = 0.f;
                if (t - lo < keep) {
                    const float rho = ratio_exp(p.logp_new[t] - p.logp_old[t]);
                    const float u = rho * p.adv[t], c = clampf(rho, p.ratio_lo, p.ratio_hi) * p.adv[t];
                    const bool unclipped = u <= c, undefined = u != u;
                    sums[0] += (double)(undefined ? u : fminf(u, c));
                    sums[2] += (double)rho;
                    sums[3] += (!unclipped && !undefined) ? 1.0 : 0.0;
                    g = undefined ? u : unclipped ? pol_coef * u : 0.f;
                }
                if (kGrad) gp.grad_logp[t] = g;
            }
            if (has_val) {
                float g = 0.f;
                if (fin) {
                    const float d0 = p.v_new[t] - p.ret[t];
                    const float d1 = clampf(p.v_new[t], p.v_old[t] - p.xi_low, p.v_old[t] + p.xi_high) - p.ret[t];
                    const bool unclipped = d0 * d0 >= d1 * d1, undefined = value_undefined(d0, d1, p.v_old[t]);
                    sums[1] += (double)(undefined ? __builtin_nanf("") : fmaxf(d0 * d0, d1 * d1));
                    sums[4] += (!unclipped && !undefined) ? 1.0 : 0.0;
                    g = undefined ? __builtin_nanf("") : unclipped ? val_coef * d0 : 0.f;
                }
                if (kGrad) gp.grad_v[t] = g;
            }
        }
    }
    block_sums(sums, s_red);
    if (tid == 0) {
        double tot[kGradSums];
#pragma unroll
        for (int q = 0; q < kGradSums; ++q) tot[q] = block_sum<kGradSums, kWaves>(s_red, q);
        if (out) write_losses(out, tot[0], tot[1], np, nv);
        if (stats) {
            stats->ratio_mean = np > 0 ? (float)(tot[2] / (double)np) : 0.f;
            stats->policy_clip_frac = np > 0 ? (float)(tot[3] / (double)np) : 0.f;
            stats->value_clip_frac = nv > 0 ? (float)(tot[4] / (double)nv) : 0.f;
            stats->reserved = 0.f;
            stats->n_policy_clipped = (long long)tot[3];
            stats->n_value_clipped = (long long)tot[4];
        }
    }
}

// Whether no workgroup of so many has more tokens than fp32 counts one by one (SumWords: the clipped ones).
constexpr bool countable(int64_t frames, int groups) { return (frames + groups - 1) / groups * (4 * kLossThreads) <= 1 << 24; }
static_assert(countable(INT32_MAX / (4 * kLossThreads) + 1, kGradGroups), "the largest batch, by the grid that counts");

// Workgroups of the persistent grids.  Nothing depends on all of them being resident at once: only the
// workgroup dispatched last waits, and only for workgroups dispatched before it.
static int loss_groups(int64_t n_resp, bool grad) {
    const int64_t frames = (n_resp + 4 * kLossThreads - 1) / (4 * kLossThreads);    // work items
    int groups = grad ? kGradGroups : kLossGroups;
#ifdef TPPO_TUNING
    if (const char* e = getenv("TPPO_LOSS_GROUPS")) {
        const int forced = atoi(e);
        if (forced >= 1 && forced <= kFinishGroups && countable(frames, forced)) groups = forced;
    }
#endif
    return frames < groups ? (int)frames : groups;
}

// Whether workgroups fetch the metadata of frames with more than two sequences (MoreSeqs).  Where a frame holds more of them
// than they fetch in one go, on the average, the fetch is one more trip before the walk that most tokens need all the same: us,
// fetching -> not, losses / derivatives: 1.0 M windows of one token 18.3 -> 15.6 / 22.9 -> 21.0;  50 000 of two 10.5 -> 9.0 / 13.3 -> 11.9;
// 10 000 of 100 tokens and 300 empty ones after each 15.4 -> 14.3 / 21.0 -> 19.3.  Below: 20 000 of eight tokens, an empty one
// after each, 8.0 (8.9) / 11.3 (12.1).  (All with sums through shuffles, on both sides.)
// (A workgroup fetches a sequence and has four tokens for each of its threads.)
static bool loss_fetches(int64_t B, int64_t n_resp) { return 4 * B < n_resp; }

// a grid of few workgroups, a frame each
static bool loss_few(int groups, int64_t n_resp) { return groups <= kFewGroups && n_resp <= (int64_t)groups * 4 * kLossThreads; }

// checks shared by the forward and the backward entry point; on TPPO_OK `plan` points at a plan of this layout
static int loss_prepare(int n_pol_ptr, int n_val_ptr, const int32_t* resp_off, const int32_t* keep_len,
                        const int32_t* done, int64_t B, int64_t n_resp, float eps_low, float eps_high, float xi_low,
                        float xi_high, void* workspace, size_t workspace_bytes, void*& plan, bool& empty,
                        int32_t* status, hipStream_t s) {
    if (B < 0 || n_resp < 0 || n_resp > INT32_MAX - kTileTokens || B > INT32_MAX / 4) return TPPO_ERR_SIZE;
    if (!(eps_low >= 0.f) || !(eps_high >= 0.f) || !(xi_low >= 0.f) || !(xi_high >= 0.f)) return TPPO_ERR_PARAM;
    if ((n_pol_ptr != 0 && n_pol_ptr != 3) || (n_val_ptr != 0 && n_val_ptr != 3)) return TPPO_ERR_NULL;
    if (B > 0 && (!resp_off || !keep_len || !done)) return TPPO_ERR_NULL;
    if (n_resp > 0 && B == 0) return TPPO_ERR_SIZE;
    if (plan_max_tiles(n_resp, B) > INT32_MAX / 8) return TPPO_ERR_SIZE;
    empty = n_resp == 0 || (n_pol_ptr == 0 && n_val_ptr == 0);
    if (plan) {
        if (!is_aligned(plan, 256)) return TPPO_ERR_WORKSPACE;
    } else {
        if (!workspace || !is_aligned(workspace, 256) ||
            workspace_bytes < plan_bytes_for(plan_max_tiles(n_resp, B)))
            return TPPO_ERR_WORKSPACE;
        if (!empty && n_resp >= 4 && launch_plan_build(resp_off, keep_len, done, B, n_resp, plan_max_tiles(n_resp, B), workspace, status, s) != TPPO_OK)
            return TPPO_ERR_LAUNCH;
        plan = workspace;
    }
    return TPPO_OK;
}

static void fill_params(LossParams& p, const float* logp_new, const float* logp_old, const float* adv,
                        const float* v_new, const float* v_old, const float* ret, const int32_t* resp_off,
                        const int32_t* keep_len, const int32_t* done, void* plan, int32_t* status, int64_t B, int64_t n_resp, float eps_low,
                        float eps_high, float xi_low, float xi_high) {
    p.logp_new = logp_new; p.logp_old = logp_old; p.adv = adv;
    p.v_new = v_new; p.v_old = v_old; p.ret = ret;
    p.resp_off = resp_off; p.keep_len = keep_len; p.done = done;
    p.plan = plan; p.status = status;
    p.B = (int)B; p.n_resp = (int)n_resp;
    p.tag = next_call_tag();
    p.ratio_lo = 1.f - eps_low; p.ratio_hi = 1.f + eps_high;
    p.xi_low = xi_low; p.xi_high = xi_high;
    p.all_ahead = B <= kLossThreads;
}

}  // namespace tppo

extern "C" size_t tppo_ppo_losses_workspace_bytes(int64_t n_resp, int64_t B) {
    if (n_resp < 0 || B < 0) return 256;
    return tppo::plan_bytes_for(tppo::plan_max_tiles(n_resp, B));
}

extern "C" int tppo_ppo_losses(const float* logp_new, const float* logp_old, const float* adv,
                               const float* v_new, const float* v_old, const float* ret,
                               const int32_t* resp_off, const int32_t* keep_len,
                               const int32_t* done, int64_t B, int64_t n_resp, float eps_low,
                               float eps_high, float xi_low, float xi_high, tppo_loss_out* out,
                               void* workspace, size_t workspace_bytes, void* plan, int32_t* status,
                               void* stream) {
    using namespace tppo;
    if (!out) return TPPO_ERR_NULL;
    const int n_pol_ptr = (logp_new != nullptr) + (logp_old != nullptr) + (adv != nullptr);
    const int n_val_ptr = (v_new != nullptr) + (v_old != nullptr) + (ret != nullptr);
    hipStream_t s = static_cast<hipStream_t>(stream);
    bool empty = false;
    const int rc = loss_prepare(n_pol_ptr, n_val_ptr, resp_off, keep_len, done, B, n_resp, eps_low, eps_high, xi_low,
                                xi_high, workspace, workspace_bytes, plan, empty, status, s);
    if (rc != TPPO_OK) return rc;
    if (empty) {
        hipLaunchKernelGGL(loss_empty_kernel, dim3(1), dim3(64), 0, s, out, (tppo_loss_stats*)nullptr);
        return launch_result();
    }
    if (n_resp < 4) {
        GradParams gp = {};
        fill_params(gp.fwd, logp_new, logp_old, adv, v_new, v_old, ret, resp_off, keep_len, done, plan, status, B, n_resp,
                    eps_low, eps_high, xi_low, xi_high);
        hipLaunchKernelGGL(loss_tiny_kernel<false>, dim3(1), dim3(256), 0, s, gp, resp_off, out, (tppo_loss_stats*)nullptr);
        return launch_result();
    }
    LossParams p;
    fill_params(p, logp_new, logp_old, adv, v_new, v_old, ret, resp_off, keep_len, done, plan, status, B, n_resp, eps_low,
                eps_high, xi_low, xi_high);
    const int groups = loss_groups(n_resp, false);
    hipLaunchKernelGGL((!loss_fetches(B, n_resp) ? loss_kernel<false, false> : loss_few(groups, n_resp) ? loss_kernel<true, true> : loss_kernel<true, false>),
                       dim3(groups), dim3(kLossThreads), 0, s, p, out);
    return launch_result();
}

extern "C" size_t tppo_ppo_losses_backward_workspace_bytes(int64_t n_resp, int64_t B) {
    return tppo_ppo_losses_workspace_bytes(n_resp, B);
}

extern "C" int tppo_ppo_losses_backward(const float* logp_new, const float* logp_old, const float* adv,
                                        const float* v_new, const float* v_old, const float* ret,
                                        const int32_t* resp_off, const int32_t* keep_len,
                                        const int32_t* done, int64_t B, int64_t n_resp, float eps_low,
                                        float eps_high, float xi_low, float xi_high, float policy_scale,
                                        float value_scale, int64_t policy_denominator,
                                        int64_t value_denominator, float* grad_logp, float* grad_v,
                                        tppo_loss_out* out, tppo_loss_stats* stats, void* workspace,
                                        size_t workspace_bytes, void* plan, int32_t* status, void* stream) {
    using namespace tppo;
    if (!(policy_scale == policy_scale) || !(value_scale == value_scale)) return TPPO_ERR_PARAM;
    const int n_pol_ptr = (logp_new != nullptr) + (logp_old != nullptr) + (adv != nullptr);
    const int n_val_ptr = (v_new != nullptr) + (v_old != nullptr) + (ret != nullptr);
    const bool halves_ok = (n_pol_ptr == 0 || n_pol_ptr == 3) && (n_val_ptr == 0 || n_val_ptr == 3);
    if (halves_ok && ((n_pol_ptr == 3) != (grad_logp != nullptr) || (n_val_ptr == 3) != (grad_v != nullptr)))
        return TPPO_ERR_NULL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    bool empty = false;
    const int rc = loss_prepare(n_pol_ptr, n_val_ptr, resp_off, keep_len, done, B, n_resp, eps_low, eps_high, xi_low,
                                xi_high, workspace, workspace_bytes, plan, empty, status, s);
    if (rc != TPPO_OK) return rc;
    if (empty) {
        if (out || stats) hipLaunchKernelGGL(loss_empty_kernel, dim3(1), dim3(64), 0, s, out, stats);
        return launch_result();
    }
    GradParams gp;
    fill_params(gp.fwd, logp_new, logp_old, adv, v_new, v_old, ret, resp_off, keep_len, done, plan, status, B, n_resp, eps_low,
                eps_high, xi_low, xi_high);
    gp.grad_logp = grad_logp; gp.grad_v = grad_v;
    gp.policy_scale = policy_scale; gp.value_scale = value_scale;
    gp.policy_denominator = policy_denominator; gp.value_denominator = value_denominator;
    if (n_resp < 4) {
        hipLaunchKernelGGL(loss_tiny_kernel<true>, dim3(1), dim3(256), 0, s, gp, resp_off, out, stats);
        return launch_result();
    }
    const int groups = loss_groups(n_resp, true);
    hipLaunchKernelGGL((!loss_fetches(B, n_resp) ? loss_grad_kernel<false, false> : loss_few(groups, n_resp) ? loss_grad_kernel<true, true> : loss_grad_kernel<true, false>),
                       dim3(groups), dim3(kLossThreads), 0, s, gp, out, stats);
    return launch_result();
}
