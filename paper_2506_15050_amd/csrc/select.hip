// tppo_select: token filter of Sec. 3.2 as a segmented compaction: per-sequence
// window / keep lengths, their prefix sums (resp_off, sel_off), the counts, then
// (row, target id, response-packed index) of every kept token and, if the caller
// wants one, the work plan of the response-packed domain (plan.h) that tppo_egae*
// and the loss entry points take.
//   up to kOneLaunchSeqs sequences: ONE launch.  Every workgroup works out all
//            lengths and prefix sums for itself, in LDS (one sequence per thread),
//            then plays its part: the small outputs and the plan's list, or a
//            share of the kept tokens and of the plan's words to zero;
//   more:    two.  One workgroup per 1024 sequences writes the lengths and prefix
//            sums and a list of tiles of the compact output (<= 1024 kept tokens of
//            one sequence each); then the plan's builders and the workgroups that
//            walk the tile list, side by side.
// Launches and the chains of dependent loads inside them are what this costs; only beyond some ten million tokens do
// the bytes written count.  Prefix sums go by data-parallel moves, a wavefront's totals by a lane each, and two workgroups of the one
// launch fit a CU: through shuffles and a loop over the wavefronts, one workgroup to a CU (the second half of 512 began when the first
// had ended) the filter took, us: 126 tokens in 3 sequences 4.9 (now 3.6), 49 K in 100 5.2 (4.1), 571 K in 1000 6.4 (5.1), 2.3 M in 512
// 11.5 (7.5), 872 K in 1500 13.3 (9.9).  Scan, plan and fill as three launches, 2.4 M tokens in 512 sequences: 29 us (7.5); 40 M
// tokens in 8704 sequences: 111 (53, 278 MB of indices).
#include "plan_build.h"

namespace tppo {

constexpr int kScanThreads = 1024;
constexpr int kOneLaunchSeqs = kScanThreads;
// Sequences before its range whose metadata a thread of the scan asks for at a time.  One by one each is a round trip: the scan of
// 8704 sequences, us, with 1 / 4 / 8: 12.0 / 10.4 / 9.8 (0.3 of each from keeping the thread's own sequence in registers).  None
// is asked for beyond the range's beginning: asked for in vain (the last one over and over) 8704, 3000 and 30 000 sequences take
// 8.2 / 7.0 / 12.4, so 7.8 / 6.5 / 12.0; one by one 9.5 / 6.7 / 12.1.
constexpr int kScanAhead = 8;
constexpr int kListParts = 8;                                   // workgroups for the list of more than 128 sequences (plan_build.h)
constexpr int kQuarter = kTileTokens / 4;                        // threads that share a tile of the compact list, four tokens each
// Workgroups on the chip at once, two on each of its 256 CUs.  (This and the lines below are fixed for the whole chip: a partition of it
// gets the same results from grids that are not tuned for it.)
constexpr int kFillMaxGroups = 512;
// Those of the second launch that walk the compact tile list, four tiles a turn.  512 of them, one turn 8 MB on from the last, are slower
// than fewer or more; the whole filter, us, 256 / 320 / 384 / 448 / 512 / 768 / 1024: 40 M tokens in 8704 sequences 61.1 / 57.2 / 54.9 / 55.2 /
// 61.9 / 56.1 / 54.3, 14 M in 3000 31.2 / 30.0 / 29.6 / 30.0 / 31.3 / 29.6 / 30.0.  Four consecutive tokens a thread, 16-byte stores: 53.3 and 29.6 with
// 384 (non-temporal ones: 82.9, 34.7).
constexpr int kWalkGroups = 384;
// The one launch's workers: beyond kManyTurns turns of all of them a workgroup to each CU stores faster than two, the whole filter, us,
// two -> one: 18 M tokens in 400 sequences 30.7 -> 26.2, in 1024 30.8 -> 29.2;  37 M in 800 60.2 -> 52.5;  8.2 M 16.7 (16.8);  7.5 M 15.7 (16.5);  2.3 M
// 7.5 (9.4).  (In turns of their own, 4 MB apart, 256 workgroups take 31.5, 34.5 and 62.9; each its own range 26.6, 29.6 and 62.2.)
constexpr int kManyTurns = 5, kManyGroups = 256;
static_assert(kScanThreads == kBuildThreads, "the same workgroups scan and build");
static_assert(4 * kQuarter == kBuildThreads, "a workgroup of the second launch walks four tiles at a time");

struct Sums { int win, keep, val, tiles; };     // window / kept / value tokens, tiles of the compact output

__device__ __forceinline__ Sums add4(Sums a, Sums b) {
    return {a.win + b.win, a.keep + b.keep, a.val + b.val, a.tiles + b.tiles};
}

__device__ __forceinline__ Sums prefix4(Sums a) {
    return {wave_prefix(a.win), wave_prefix(a.keep), wave_prefix(a.val), wave_prefix(a.tiles)};
}

__device__ __forceinline__ Sums lane_of(Sums a, int lane) {
    return {__builtin_amdgcn_readlane(a.win, lane), __builtin_amdgcn_readlane(a.keep, lane), __builtin_amdgcn_readlane(a.val, lane),
            __builtin_amdgcn_readlane(a.tiles, lane)};
}
__device__ __forceinline__ Sums lane63(Sums a) { return lane_of(a, kWave - 1); }

static inline int64_t select_max_tiles(int64_t capacity, int64_t B) { return capacity / kTileTokens + B + 1; }

struct SeqWords { int lo, hi, ctx, done; };      // a sequence's metadata as it stands in memory

__device__ __forceinline__ SeqWords words_of(const int32_t* __restrict__ cu_seqlens, const int32_t* __restrict__ ctx_len,
                                             const int32_t* __restrict__ done, int i) {
    return {cu_seqlens[i], cu_seqlens[i + 1], ctx_len[i], done[i]};
}

// window / keep lengths of a sequence (a bad layout counts as an empty window and sets the status bit)
__device__ __forceinline__ Sums lengths_of(SeqWords x, int n_tok, int tail_drop, int32_t* status) {
    int win = x.hi - x.lo - x.ctx;
    if (x.ctx < 1 || win < 0 || x.lo < 0 || x.hi > n_tok) {
        if (status) set_status(status, TPPO_STATUS_BAD_LAYOUT);
        win = 0;
    }
    const bool fin = x.done != 0;
    const int keep = fin ? win : max(win - tail_drop, 0);
    return {win, keep, fin ? win : 0, tiles_of(keep)};
}

// `parts` workgroups share the sequences (one up to a few thousand of them): workgroup g owns a contiguous
// range and, inside it, thread t a contiguous block, so there is one workgroup-wide prefix sum whatever B is:
// pass A adds up the block, the scan gives the block's starting offsets, pass B re-reads the (cache-resident)
// metadata and writes the per-sequence outputs and tile descriptors.  Where its range starts a workgroup
// finds out by adding up, by itself, the lengths of all sequences before the range.
__global__ __launch_bounds__(kScanThreads) void select_scan_kernel(
    const int32_t* __restrict__ cu_seqlens, const int32_t* __restrict__ ctx_len,
    const int32_t* __restrict__ done, int B, int n_tok, int tail_drop, int parts,
    int32_t* __restrict__ resp_off, int32_t* __restrict__ sel_off,
    int32_t* __restrict__ keep_len, int64_t* __restrict__ counts, Tile* __restrict__ tiles,
    int tile_cap, int32_t* __restrict__ n_tiles, int32_t* status) {
    __shared__ Sums wave_tot[2][kScanThreads / kWave];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int part = blockIdx.x;
    const int range = (B + parts - 1) / parts;
    const int p_begin = min(part * range, B), p_end = min(p_begin + range, B);
    const int per = (p_end - p_begin + kScanThreads - 1) / kScanThreads;
    const int i_begin = min(p_begin + tid * per, p_end), i_end = min(i_begin + per, p_end);
    Sums mine = {0, 0, 0, 0}, ahead = {0, 0, 0, 0};
    const SeqWords first = words_of(cu_seqlens, ctx_len, done, min(i_begin, B - 1));
    for (int base = 0; base < p_begin; base += kScanAhead * kScanThreads) {
        const int i0 = base + tid;
        SeqWords x[kScanAhead];
#pragma unroll
        for (int k = 0; k < kScanAhead; ++k)
            if (base + k * kScanThreads < p_begin) x[k] = words_of(cu_seqlens, ctx_len, done, min(i0 + k * kScanThreads, p_begin - 1));
#pragma unroll
        for (int k = 0; k < kScanAhead; ++k)
            if (i0 + k * kScanThreads < p_begin) ahead = add4(ahead, lengths_of(x[k], n_tok, tail_drop, nullptr));
    }
    for (int i = i_begin; i < i_end; ++i)
        mine = add4(mine, lengths_of(i == i_begin ? first : words_of(cu_seqlens, ctx_len, done, i), n_tok, tail_drop, status));
    const Sums inc = prefix4(mine), before = prefix4(ahead);
    if (lane == kWave - 1) {
        wave_tot[0][wave] = inc;
        wave_tot[1][wave] = before;
    }
    __syncthreads();
    // the wavefronts' totals, a lane each: what comes before my wavefront, and all there is
    constexpr int kWaves = kScanThreads / kWave;
    const Sums none = {0, 0, 0, 0};
    const Sums wave_inc = prefix4(lane < kWaves ? wave_tot[0][lane] : none), all_before = lane63(prefix4(lane < kWaves ? wave_tot[1][lane] : none));
    const Sums total = add4(lane63(wave_inc), all_before);
    Sums run = {inc.win - mine.win, inc.keep - mine.keep, inc.val - mine.val, inc.tiles - mine.tiles};
    run = add4(run, all_before);
    if (wave > 0) run = add4(run, lane_of(wave_inc, wave - 1));
    if (part == 0 && tid == 0) {
        resp_off[0] = 0;
        sel_off[0] = 0;
    }
    for (int i = i_begin; i < i_end; ++i) {
        const Sums x = lengths_of(i == i_begin ? first : words_of(cu_seqlens, ctx_len, done, i), n_tok, tail_drop, nullptr);
        keep_len[i] = x.keep;
        if (tiles) emit_tiles(tiles, tile_cap, run.tiles, i, run.keep, x.keep);       // compact domain
        run = add4(run, x);
        resp_off[i + 1] = run.win;
        sel_off[i + 1] = run.keep;
    }
    if (part == parts - 1 && tid == 0) {                // the last range ends where the batch ends
        counts[0] = total.keep;
        counts[1] = total.win;
        counts[2] = total.val;
        if (n_tiles) n_tiles[0] = min(total.tiles, tile_cap);
    }
}

struct FillArgs {
    const int32_t *cu_seqlens, *ctx_len, *input_ids;
    int32_t *sel_rows, *sel_targets, *sel_resp_idx;
    int64_t capacity;
    int n_tok;
    int32_t* status;
};

// (any `m`: 4-byte alignment will do)
typedef int32_t int4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ void store_some(int32_t* dst, int64_t m, const int (&x)[4], int n) {
    if (n == 4) {
        *reinterpret_cast<int4u*>(dst + m) = int4u{x[0], x[1], x[2], x[3]};
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (e < n) dst[m + e] = x[e];
    }
}

// the ids at four packed positions, the first `some` of them wanted; run: one after the other
__device__ __forceinline__ void load_ids(const FillArgs& a, const int (&pos)[4], bool run, int some, int (&id)[4]) {
    if (run && pos[0] >= 0 && pos[0] <= a.n_tok - 4) {
        const int4u x = *reinterpret_cast<const int4u*>(a.input_ids + pos[0]);
#pragma unroll
        for (int e = 0; e < 4; ++e) id[e] = x[e];
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) id[e] = (e < some && pos[e] >= 0 && pos[e] < a.n_tok) ? a.input_ids[pos[e]] : -1;
    }
}

// Second launch of the large case.  Workgroups 0 .. parts-1 build the plan's list and workgroup `parts` counts its
// sets (none of these without a plan); the others zero the plan's words and walk the compact tile list, four
// tiles at a time.
__global__ __launch_bounds__(kBuildThreads) void select_fill_kernel(FillArgs a, const int32_t* __restrict__ resp_off,
                                                                    const int32_t* __restrict__ keep_len,
                                                                    const int32_t* __restrict__ done, int B,
                                                                    const Tile* __restrict__ tiles,
                                                                    const int32_t* __restrict__ n_tiles, int parts,
                                                                    int plan_cap, void* plan_raw) {
    __shared__ union {
        BuildLds build;
        SetLds sets;
    } s;
    int worker = blockIdx.x, workers = gridDim.x;
    if (plan_raw) {
        const Plan pl = plan_view(plan_raw, plan_cap);
        if (worker < parts) {
            build_list(pl, s.build, resp_off, keep_len, done, true, B, resp_off[B], worker, parts, a.status);
            return;
        }
        if (worker == parts) {
            count_sets(pl, s.sets, resp_off, keep_len, done, B);
            return;
        }
        worker -= parts + 1;
        workers -= parts + 1;
        clear_words(pl, worker, workers);
    }
    if (!tiles) return;
    const int count = *n_tiles;
    const int quarter = threadIdx.x / kQuarter, tid = threadIdx.x % kQuarter;
    for (int w = worker * 4 + quarter; w < count; w += workers * 4) {
        const Tile t = tiles[w];
        const int i = t.seg, t0 = t.number() * kTileTokens, k = 4 * tid;
        const int64_t m = (int64_t)t.start + k;
        const int n = min(t.len() - k, 4), some = (int)max(min((int64_t)n, a.capacity - m), (int64_t)0);
        if (n <= 0) continue;
        if (some < n && m + some == a.capacity) set_status(a.status, TPPO_STATUS_CAPACITY);
        const int pos = a.cu_seqlens[i] + a.ctx_len[i] + t0 + k;     // packed position of the first of the four
        const int resp = resp_off[i] + t0 + k;
        if (a.sel_rows) store_some(a.sel_rows, m, {pos - 1, pos, pos + 1, pos + 2}, some);
        if (a.sel_targets) {
            int id[4];
            load_ids(a, {pos, pos + 1, pos + 2, pos + 3}, true, some, id);
            store_some(a.sel_targets, m, id, some);
        }
        if (a.sel_resp_idx) store_some(a.sel_resp_idx, m, {resp, resp + 1, resp + 2, resp + 3}, some);
    }
}

// The whole filter in one launch, B <= kOneLaunchSeqs.  Workgroups 0 .. parts - 1 write the plan's list, the first of them also
// the small outputs; the others zero the plan's words and write the kept tokens, four consecutive ones per thread and turn, whose
// sequence a thread finds by bisection of the offsets in LDS.
// (With 88 scalar registers, and the 16 that each wavefront has besides, a CU takes one workgroup: 2.3 M tokens 9.3 instead of 7.5.)
__global__ __launch_bounds__(kBuildThreads) __attribute__((amdgpu_num_sgpr(80))) void select_one_launch_kernel(
    FillArgs a, const int32_t* __restrict__ done, int B, int tail_drop, int32_t* __restrict__ resp_off, int32_t* __restrict__ sel_off,
    int32_t* __restrict__ keep_len, int64_t* __restrict__ counts, int parts, int plan_cap, void* plan_raw) {
    __shared__ int32_t s_resp[kOneLaunchSeqs + 1], s_sel[kOneLaunchSeqs + 1], s_aux[2][kOneLaunchSeqs];
    __shared__ int s_wave[3][kBuildWaves];
    __shared__ BuildLds s_build;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool lead = (int)blockIdx.x < parts, first = blockIdx.x == 0;
    const int worker = (int)blockIdx.x - parts, workers = (int)gridDim.x - parts;
    Sums mine = {0, 0, 0, 0};
    int first_pos = 0;
    bool fin = false;
    if (tid < B) {
        mine = lengths_of(words_of(a.cu_seqlens, a.ctx_len, done, tid), a.n_tok, tail_drop, first ? a.status : nullptr);
        first_pos = a.cu_seqlens[tid] + a.ctx_len[tid];
        fin = done[tid] != 0;
    }
    const Plan pl = plan_view(plan_raw, plan_cap);
    if (plan_raw && !lead) clear_words(pl, worker, workers);         // (while the lengths are on their way)
    int win = wave_prefix(mine.win), keep = wave_prefix(mine.keep);  // inclusive prefix sums
    const int val = wave_prefix(mine.val);
    if (lane == kWave - 1) {
        s_wave[0][wave] = win;
        s_wave[1][wave] = keep;
        s_wave[2][wave] = val;
    }
    __syncthreads();
    // the wavefronts' totals, a lane each, and what comes before mine
    const int at = min(lane, kBuildWaves - 1);
    const int wins = wave_prefix(s_wave[0][at]), keeps = wave_prefix(s_wave[1][at]);
    if (wave > 0) {
        win += __builtin_amdgcn_readlane(wins, wave - 1);
        keep += __builtin_amdgcn_readlane(keeps, wave - 1);
    }
    if (tid == 0) s_resp[0] = s_sel[0] = 0;
    if (tid < B) {
        s_resp[tid + 1] = win;
        s_sel[tid + 1] = keep;
        s_aux[0][tid] = lead ? mine.keep : first_pos;
        s_aux[1][tid] = fin;
    }
    __syncthreads();
    const int n_kept = s_sel[B];
    if (lead) {
        if (first && tid < B) {
            keep_len[tid] = mine.keep;
            resp_off[tid + 1] = win;
            sel_off[tid + 1] = keep;
        }
        if (first && tid == 0) {
            resp_off[0] = 0;
            sel_off[0] = 0;
            long long n_val = 0;
#pragma unroll
            for (int w = 0; w < kBuildWaves; ++w) n_val += s_wave[2][w];
            counts[0] = n_kept;
            counts[1] = s_resp[B];
            counts[2] = n_val;
            if ((a.sel_rows || a.sel_targets || a.sel_resp_idx) && n_kept > a.capacity)
                set_status(a.status, TPPO_STATUS_CAPACITY);
            if (plan_raw) {
                pl.hdr->n_policy = n_kept;
                pl.hdr->n_value = n_val;
                pl.hdr->has_sets = 1;
            }
        }
        if (plan_raw)
            build_list_by_level(pl, s_build, (const int32_t*)s_resp, (const int32_t*)s_aux[0], (const int32_t*)s_aux[1], B,
                                s_resp[B], (int)blockIdx.x, parts, a.status);
        return;
    }
    if (!a.sel_rows && !a.sel_targets && !a.sel_resp_idx) return;
    const int64_t n = min((int64_t)n_kept, a.capacity);
    // Many turns are taken by a workgroup to a CU, the places of the others after its own (kManyTurns).
    const int64_t turn = (int64_t)workers * kBuildThreads * 4;
    const int active = n > kManyTurns * turn ? min(workers, kManyGroups) : workers;
    if (worker >= active) return;
    for (int place = worker; place < workers; place += active) {
        for (int64_t m = ((int64_t)place * kBuildThreads + tid) * 4; m < n; m += turn) {
            int lo = 0, hi = B - 1;                                      // the last sequence that begins at or before m
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (s_sel[mid] <= m) lo = mid; else hi = mid - 1;
            }
            const int some = (int)min(n - m, (int64_t)4);
            int pos[4], resp[4], id[4];
            const bool run = m + 4 <= s_sel[lo + 1];                     // all four in one sequence
            if (run) {
                const int t = (int)m - s_sel[lo];
                const int p0 = s_aux[0][lo] + t, r0 = s_resp[lo] + t;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    pos[e] = p0 + e;
                    resp[e] = r0 + e;
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    while (lo < B - 1 && s_sel[lo + 1] <= (int)m + e) ++lo;
                    const int t = (int)m + e - s_sel[lo];
                    pos[e] = s_aux[0][lo] + t;
                    resp[e] = s_resp[lo] + t;
                }
            }
            if (a.sel_targets) {
                load_ids(a, pos, run, some, id);
                store_some(a.sel_targets, m, id, some);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) pos[e] -= 1;
            if (a.sel_rows) store_some(a.sel_rows, m, pos, some);
            if (a.sel_resp_idx) store_some(a.sel_resp_idx, m, resp, some);
        }
    }
}

// The one launch's grid.  Its workers and the list's workgroups are on the chip together: one beyond the kFillMaxGroups places
// waits until another has ended and goes through the whole chain, metadata to prefix sums, after it.
static int list_parts(bool plan, int64_t B) { return plan && B > 2 * kWave ? kListParts : 1; }
static int one_launch_workers(int64_t most, int parts) { return (int)(most < kFillMaxGroups - parts ? most : kFillMaxGroups - parts); }

}  // namespace tppo

extern "C" size_t tppo_select_workspace_bytes(int64_t B, int64_t capacity) {
    if (B < 0 || capacity < 0) return 256;
    return tppo::round_up((size_t)tppo::select_max_tiles(capacity, B) * sizeof(tppo::Tile), 256) + 256;
}

extern "C" int tppo_select(const int32_t* cu_seqlens, const int32_t* ctx_len, const int32_t* done,
                           const int32_t* input_ids, int64_t B, int64_t n_tok, int32_t tail_drop,
                           int32_t* resp_off, int32_t* sel_off, int32_t* keep_len,
                           int32_t* sel_rows, int32_t* sel_targets, int32_t* sel_resp_idx,
                           int64_t capacity, int64_t* counts, void* workspace, size_t workspace_bytes,
                           void* plan, size_t plan_bytes, int32_t* status, void* stream) {
    using namespace tppo;
    if (B < 0 || n_tok < 0 || capacity < 0 || B > INT32_MAX / 4 || n_tok > INT32_MAX) return TPPO_ERR_SIZE;
    if (tail_drop < 0) return TPPO_ERR_PARAM;
    if (!cu_seqlens || !resp_off || !sel_off || !counts) return TPPO_ERR_NULL;
    if (B > 0 && (!ctx_len || !done || !keep_len)) return TPPO_ERR_NULL;
    if (sel_targets && !input_ids) return TPPO_ERR_NULL;
    const bool want_fill = (sel_rows || sel_targets || sel_resp_idx) && B > 0 && capacity > 0;
    // the list covers every kept token, also those beyond `capacity` (they are reported, not written)
    const int64_t list_tokens = capacity < n_tok ? n_tok : capacity;
    const int64_t cap64 = select_max_tiles(list_tokens, B);
    if (cap64 > INT32_MAX / 4) return TPPO_ERR_SIZE;
    if (want_fill && (!workspace || !is_aligned(workspace, 256) ||
                      workspace_bytes < tppo_select_workspace_bytes(B, list_tokens)))
        return TPPO_ERR_WORKSPACE;
    // a plan is sized for the largest response-packed domain this batch can have: n_resp <= n_tok
    const int64_t plan_cap = plan_max_tiles(n_tok, B);
    if (plan && (!is_aligned(plan, 256) || plan_bytes < plan_bytes_for(plan_cap) || plan_cap > INT32_MAX / 8))
        return TPPO_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    FillArgs a = {cu_seqlens, ctx_len, input_ids, nullptr, nullptr, nullptr, capacity, (int)n_tok, status};
    if (want_fill) {
        a.sel_rows = sel_rows;
        a.sel_targets = sel_targets;
        a.sel_resp_idx = sel_resp_idx;
    }
    // enough workgroups that zero or fill to keep every CU busy, each with a few turns on a large batch
    const int64_t clear = plan ? (plan_words(plan_cap) + kBuildThreads * 8 - 1) / (kBuildThreads * 8) : 0;
    const int64_t fill = want_fill ? (n_tok + kBuildThreads * 4 - 1) / (kBuildThreads * 4) : 0;
    const int64_t most = clear > fill ? clear : fill;
    if (B <= kOneLaunchSeqs) {
        const int parts = list_parts(plan != nullptr, B), workers = one_launch_workers(most, parts);
        hipLaunchKernelGGL(select_one_launch_kernel, dim3(parts + workers), dim3(kBuildThreads), 0, s, a, done, (int)B,
                           (int)tail_drop, resp_off, sel_off, keep_len, counts, parts, (int)plan_cap, plan);
        return launch_result();
    }
    Tile* tiles = want_fill ? static_cast<Tile*>(workspace) : nullptr;
    int32_t* n_tiles = want_fill ? reinterpret_cast<int32_t*>(static_cast<char*>(workspace) +
                                                              round_up((size_t)cap64 * sizeof(Tile), 256))
                                 : nullptr;
    const int parts = build_parts(B), workers = (int)(most < kWalkGroups ? most : kWalkGroups);
    hipLaunchKernelGGL(select_scan_kernel, dim3(parts), dim3(kScanThreads), 0, s, cu_seqlens, ctx_len,
                       done, (int)B, (int)n_tok, (int)tail_drop, parts, resp_off, sel_off, keep_len, counts,
                       tiles, (int)cap64, n_tiles, status);
    if (launch_result() != TPPO_OK) return TPPO_ERR_LAUNCH;
    const int groups = (plan ? parts + 1 : 0) + workers;             // n_resp is known on the device only
    if (groups == 0) return TPPO_OK;
    hipLaunchKernelGGL(select_fill_kernel, dim3(groups), dim3(kBuildThreads), 0, s, a, resp_off, keep_len, done, (int)B,
                       tiles, n_tiles, parts, (int)plan_cap, plan);
    return launch_result();
}
