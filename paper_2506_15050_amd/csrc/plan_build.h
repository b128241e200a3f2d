// Device side of building a work plan (plan.h), shared by the kernels that do it: plan.hip's, from offsets in
// memory, and select.hip's, from offsets it has just computed.
#pragma once
#include "plan.h"

namespace tppo {

constexpr int kBuildWaves = kBuildThreads / kWave;

// (resp_off: int32, in memory or in LDS)
template <class Ints>
__device__ __forceinline__ int window_of(Ints resp_off, int i, int n_resp, int& lo, int32_t* status) {
    lo = resp_off[i];
    const int hi = resp_off[i + 1];
    if (lo < 0 || hi < lo || hi > n_resp) {
        if (status) set_status(status, TPPO_STATUS_BAD_LAYOUT);
        return 0;
    }
    return hi - lo;
}

// Tiles are cut at multiples of kTileTokens of the response-packed INDEX, not of the position inside the
// sequence: every tile but a sequence's first and last is then a 4 KiB-aligned block of each array (given
// aligned arrays), which is worth 10-15 % to a streaming kernel on this chip -- a wavefront's 1 KiB access
// that straddles 128-byte lines costs an extra line each time.  The price is up to one more (short) tile per
// sequence.
__host__ __device__ __forceinline__ int window_tiles(int lo, int len) {
    return len > 0 ? ((lo + len - 1) / kTileTokens) - (lo / kTileTokens) + 1 : 0;
}

// The sequence that follows [lo, end) inside the frame that holds its last token, if that frame is the sequence's to
// describe (it begins there) and goes on: skipping at most kSkipEmpty empty ones; beyond that the consumers
// look for themselves.  Looked up once per sequence, before its tiles are written: inside the loop over the tiles
// the dependent loads were a microsecond each.
constexpr int kSkipEmpty = 64;
struct NextSeq {
    int seg, end, pol_end, fin;
};
template <class Ints>
__host__ __device__ __forceinline__ NextSeq next_sequence(int seg, int lo, int end, Ints resp_off, Ints keep_len, Ints done,
                                                          bool sets, int B, int n_resp) {
    NextSeq x = {seg, end, end, 0};
    const int frame = (end - 1) & ~(kTileTokens - 1);
    if (frame < lo || end >= frame + kTileTokens || end >= n_resp) return x;
    int j = seg + 1;
    for (int step = 0; step < kSkipEmpty && j < B && resp_off[j + 1] <= end; ++step) ++j;
    if (j < B && resp_off[j] == end && resp_off[j + 1] > end && resp_off[j + 1] <= n_resp) {
        const int len = resp_off[j + 1] - end;
        x.seg = j;
        x.end = end + len;
        x.pol_end = sets ? end + min(max((int)keep_len[j], 0), len) : end;
        x.fin = (sets && done[j] != 0) ? 1 : 0;
    }
    return x;
}

// The tile that begins a frame describes the frame.
__host__ __device__ __forceinline__ void note_frame(const Plan& pl, const Tile& d, int lo, int len, bool sets, int keep, bool fin,
                                                    const NextSeq& next) {
    if ((d.start & (kTileTokens - 1)) != 0) return;
    const int f = d.start / kTileTokens;
    if (f >= pl.cap) return;
    const int end = lo + len;
    FrameDesc x = {d.seg, end, sets ? lo + min(max(keep, 0), len) : lo, fin ? 1 : 0, d.seg, end, end, 0};
    if (d.after == 0) {
        x.seg2 = next.seg;
        x.end2 = next.end;
        x.pol_end2 = next.pol_end;
        x.fin2 = next.fin;
    }
    pl.frames[f] = x;
}

__host__ __device__ __forceinline__ Tile make_tile(int seg, int lo, int len, int tiles, int after) {
    const int c = tiles - 1 - after;
    const int block = lo / kTileTokens + c;                             // which aligned block of the arrays
    const int first = max(lo, block * kTileTokens), last = min(lo + len, (block + 1) * kTileTokens);
    Tile d;
    d.start = first;
    d.pos_len = (c << kTileShift) | (last - first - 1);
    d.seg = seg;
    d.after = after;
    return d;
}

// One kBuildThreads-sized workgroup's part of the list: workgroup `part` of `parts` owns a contiguous range of the
// sequences and, inside it, thread t a contiguous block.  A tile of level l goes to
//   (tiles of lower levels, whole batch) + (level-l tiles of the sequences before the range)
//   + (level-l tiles of the range's wavefronts before mine) + (its rank inside the wavefront).
// Every builder counts the first two terms by itself, from offsets that sit in the cache -- cheaper than a
// second launch.  All counting is by ballot, level by level, in loops that run as deep as the longest
// sequence the wavefront is looking at: the code stays small (a kernel that runs once per batch pays for
// every instruction-cache line it touches; the fully unrolled form of this one took 20 us on 32 sequences)
// and short batches cost little.  Lane l holds the counter of level l (lane kLevels: of the tiles beyond the sorted
// levels).  Inside a level the order is whatever the ballots give; only the level order matters.
struct BuildLds {
    // per wavefront and level: tiles of the whole batch [0], of the sequences before my range [1], of my range [2]
    int count[3][kBuildWaves][kLevels + 1];
    int sum[2][kLevels + 1];
    int first[kLevels + 1];                                // list position of the range's first tile of a level
    int total;
};
static_assert(kLevels < kWave, "one lane per level and one for the tiles beyond");
static_assert(kBuildWaves == 16, "a row of 16 lanes holds a level's groups");

template <class Ints>
__device__ __forceinline__ void build_list(const Plan& pl, BuildLds& s, Ints resp_off, Ints keep_len, Ints done, bool sets,
                                           int B, int n_resp, int part, int parts, int32_t* status) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, cap = pl.cap;
    const int range = (B + parts - 1) / parts;
    const int p_begin = min(part * range, B), p_end = min(p_begin + range, B);
    const int per = (p_end - p_begin + kBuildThreads - 1) / kBuildThreads;
    const int i_begin = min(p_begin + tid * per, p_end), i_end = min(i_begin + per, p_end);
    int lo = 0;
    const unsigned long long below = (1ull << lane) - 1;          // lanes before mine
    auto count_levels = [&](int& counter, int tiles) {
        const int deepest = wave_max(tiles);
        for (int l = 0; l < min(deepest, kLevels); ++l) {
            const int c = __popcll(__ballot(tiles > l));
            counter += lane == l ? c : 0;
        }
        if (deepest > kLevels) {                                    // tiles beyond the sorted levels
            const int extra = __builtin_amdgcn_readlane(wave_prefix(max(tiles - kLevels, 0)), kWave - 1);
            counter += lane == kLevels ? extra : 0;
        }
    };
    int c_all = 0, c_ahead = 0, c_mine = 0;
    // my range: thread t owns sequences i_begin .. i_end - 1; the wavefront handles one of each at a time
    for (int k = 0; k < per; ++k) {
        const int i = i_begin + k;
        int tiles = 0;
        if (i < i_end) {
            const int len = window_of(resp_off, i, n_resp, lo, status);
            tiles = window_tiles(lo, len);
        }
        count_levels(c_mine, tiles);
    }
    if (parts == 1) {
        c_all = c_mine;
    } else {                            // whole batch and the sequences before my range: every wavefront its share, strided
        for (int i0 = wave * kWave; i0 < B; i0 += kBuildThreads) {
            const int i = i0 + lane;
            int tiles = 0;
            if (i < B) {
                const int len = window_of(resp_off, i, n_resp, lo, nullptr);
                tiles = window_tiles(lo, len);
            }
            count_levels(c_all, tiles);
            if (i0 < p_begin) count_levels(c_ahead, i < p_begin ? tiles : 0);
        }
    }
    if (lane <= kLevels) {
        s.count[0][wave][lane] = c_all;
        s.count[1][wave][lane] = c_ahead;
        s.count[2][wave][lane] = c_mine;
    }
    __syncthreads();
    if (tid < 2 * (kLevels + 1)) {                                  // totals over the wavefronts
        const int which = tid / (kLevels + 1), l = tid % (kLevels + 1);
        int sum = 0;
#pragma unroll
        for (int w = 0; w < kBuildWaves; ++w) sum += s.count[which][w][l];
        s.sum[which][l] = sum;
    }
    int at_level = 0;                                               // my wavefront's running offset inside level `lane`
    if (lane <= kLevels) {
        for (int w = 0; w < wave; ++w) at_level += s.count[2][w][lane];
    }
    __syncthreads();
    if (tid < kWave) {                                              // where each level starts for this range
        const int mine = tid <= kLevels ? s.sum[0][tid] : 0;
        const int inc = wave_prefix(mine);
        if (tid <= kLevels) s.first[tid] = inc - mine + s.sum[1][tid];
        if (tid == kLevels) s.total = inc;
    }
    __syncthreads();
    if (lane <= kLevels) at_level += s.first[lane];
    // Emission, in the same order as the count of my range.
    for (int k = 0; k < per; ++k) {
        const int i = i_begin + k;
        int tiles = 0, len = 0, keep = 0;
        bool fin = false;
        NextSeq next = {0, 0, 0, 0};
        if (i < i_end) {
            len = window_of(resp_off, i, n_resp, lo, nullptr);
            tiles = window_tiles(lo, len);
            if (sets && tiles > 0) {
                keep = keep_len[i];
                fin = done[i] != 0;
            }
            if (tiles > 0) next = next_sequence(i, lo, lo + len, resp_off, keep_len, done, sets, B, n_resp);
        }
        const int deepest = wave_max(tiles);
        for (int l = 0; l < min(deepest, kLevels); ++l) {
            const unsigned long long has = __ballot(tiles > l);
            const int at = __builtin_amdgcn_readlane(at_level, l) + __popcll(has & below);
            if (tiles > l && at < cap) {                            // (invalid offsets cannot overflow the list)
                const Tile d = make_tile(i, lo, len, tiles, l);
                pl.tiles[at] = d;
                note_frame(pl, d, lo, len, sets, keep, fin, next);
            }
            at_level += lane == l ? __popcll(has) : 0;
        }
        if (deepest > kLevels) {                                    // a sequence's deeper tiles stay together
            const int extra = max(tiles - kLevels, 0);
            const int inc = wave_prefix(extra);
            int at = __builtin_amdgcn_readlane(at_level, kLevels) + inc - extra;
            for (int l = kLevels; l < tiles; ++l, ++at) {
                if (at < cap) {
                    const Tile d = make_tile(i, lo, len, tiles, l);
                    pl.tiles[at] = d;
                    note_frame(pl, d, lo, len, sets, keep, fin, next);
                }
            }
            const int total = __builtin_amdgcn_readlane(inc, kWave - 1);
            at_level += lane == kLevels ? total : 0;
        }
    }
    if (part == parts - 1 && tid == 0) {
        const int total = s.total;
        if (total > cap) set_status(status, TPPO_STATUS_BAD_LAYOUT);
        pl.hdr->n_tiles = min(total, cap);
        pl.hdr->B = B;
        pl.hdr->n_resp = n_resp;
        pl.hdr->cap = cap;
    }
}

// The same list for up to kBuildThreads sequences whose offsets, kept lengths and flags lie in LDS, so that any wavefront can
// look at all of them: wavefronts take levels of groups of 64 sequences, one ballot and one store a lane each, and where a
// few long sequences are most of the batch, a sequence's tiles beyond the sorted levels go out 64 at a time.  A lane that
// walks down its own sequence's levels takes as long as the longest has tiles.  The whole filter, us, by the lanes' walk -> so:
// 40 sequences of up to 88 tiles 15.9 -> 9.5; 93 of up to 7 7.1 -> 6.3; beyond 128 sequences eight workgroups share the
// (level, group) pairs: 200 of up to 4 6.5 -> 5.7; 512 of up to 20 11.7 -> 10.0; 900 of up to 40 23.7 -> 16.7; 700 of up to 6 11.5 ->
// 11.5, where four workgroups take 11.7, and 11.9 if they count and place tiles beyond the sorted levels that no sequence
// has and leave other workgroups without a place on the chip (select.hip).
template <class Ints>
__device__ __forceinline__ void build_list_by_level(const Plan& pl, BuildLds& s, Ints resp_off, Ints keep_len, Ints done, int B,
                                                    int n_resp, int part, int parts, int32_t* status) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, cap = pl.cap;
    const int groups = (B + kWave - 1) / kWave;                     // of 64 sequences, at most as many as there are wavefronts
    const unsigned long long below = (1ull << lane) - 1;            // lanes before mine
    int lo = 0, len = 0;
    auto tiles_at = [&](int i, int32_t* st) {
        len = i < B ? window_of(resp_off, i, n_resp, lo, st) : 0;
        return window_tiles(lo, len);
    };
    int counter = 0, deepest = 0;                                   // lane l: group `wave`'s tiles of level l
    if (wave < groups) {
        const int tiles = tiles_at(wave * kWave + lane, part == 0 ? status : nullptr);
        deepest = wave_max(tiles);
        for (int l = 0; l < min(deepest, kLevels); ++l) {
            const int c = __popcll(__ballot(tiles > l));
            counter = lane == l ? c : counter;
        }
        if (deepest > kLevels) {                                    // tiles beyond the sorted levels
            const int extra = __builtin_amdgcn_readlane(wave_prefix(max(tiles - kLevels, 0)), kWave - 1);
            counter = lane == kLevels ? extra : counter;
        }
    }
    if (lane <= kLevels) s.count[0][wave][lane] = counter;
    __syncthreads();
    // Where each group's tiles of a level begin: 16 lanes a level for the groups, then every wavefront for itself the levels'
    // beginnings, lane l's in `level_at`.  (One wavefront going through the groups for all took half a microsecond more.)
    for (int l = tid / kBuildWaves; l <= kLevels; l += kBuildThreads / kBuildWaves) {
        const int g = tid % kBuildWaves, mine = s.count[0][g][l];
        int inc = mine;
        inc += dpp_move<kRowShr1, 0xF>(inc);
        inc += dpp_move<kRowShr2, 0xF>(inc);
        inc += dpp_move<kRowShr4, 0xF>(inc);
        inc += dpp_move<kRowShr8, 0xF>(inc);
        s.count[1][g][l] = inc - mine;
        if (g == kBuildWaves - 1) s.sum[0][l] = inc;
    }
    __syncthreads();
    const int of_level = lane <= kLevels ? s.sum[0][lane] : 0, up_to = wave_prefix(of_level), level_at = up_to - of_level;
    const int levels = __popcll(__ballot(lane < kLevels && of_level > 0)), total = __builtin_amdgcn_readlane(up_to, kWave - 1);
    for (int task = part * kBuildWaves + wave, n = levels * groups; task < n; task += parts * kBuildWaves) {
        const int l = task / groups, g = task - l * groups;
        if (s.count[0][g][l] == 0) continue;                        // (uniform)
        const int i = g * kWave + lane, tiles = tiles_at(i, nullptr);
        const int at = __builtin_amdgcn_readlane(level_at, l) + s.count[1][g][l] + __popcll(__ballot(tiles > l) & below);
        if (tiles > l && at < cap) {                                // (invalid offsets cannot overflow the list)
            const Tile d = make_tile(i, lo, len, tiles, l);
            pl.tiles[at] = d;
            NextSeq next = {0, 0, 0, 0};
            if (l == 0) next = next_sequence(i, lo, lo + len, resp_off, keep_len, done, true, B, n_resp);
            note_frame(pl, d, lo, len, true, keep_len[i], done[i] != 0, next);
        }
    }
    if (deepest > kLevels && part == parts - 1) {                       // a sequence's deeper tiles stay together
        const int i = wave * kWave + lane, tiles = tiles_at(i, nullptr), extra = max(tiles - kLevels, 0);
        const int begin = __builtin_amdgcn_readlane(level_at, kLevels) + s.count[1][wave][kLevels] + wave_prefix(extra) - extra;
        for (unsigned long long todo = __ballot(extra > 0); todo != 0; todo &= todo - 1) {
            const int j = __ffsll(todo) - 1, seq = wave * kWave + j, n = __shfl(tiles, j), from = __shfl(begin, j);
            const int seq_lo = __shfl(lo, j), seq_len = __shfl(len, j);
            for (int l = kLevels + lane; l < n; l += kWave) {
                const int mine = from + l - kLevels;
                if (mine < cap) {
                    const Tile d = make_tile(seq, seq_lo, seq_len, n, l);
                    pl.tiles[mine] = d;
                    note_frame(pl, d, seq_lo, seq_len, true, keep_len[seq], done[seq] != 0, NextSeq{0, 0, 0, 0});
                }
            }
        }
    }
    if (part == parts - 1 && tid == 0) {
        if (total > cap) set_status(status, TPPO_STATUS_BAD_LAYOUT);
        pl.hdr->n_tiles = min(total, cap);
        pl.hdr->B = B;
        pl.hdr->n_resp = n_resp;
        pl.hdr->cap = cap;
    }
}

// One workgroup: sizes of the two token sets, from the metadata alone.
struct SetLds {
    long long part[2][kBuildWaves];
};
__device__ __forceinline__ void count_sets(const Plan& pl, SetLds& s, const int32_t* resp_off, const int32_t* keep_len,
                                           const int32_t* done, int B) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    long long np = 0, nv = 0;
    if (keep_len) {
        for (int i = tid; i < B; i += kBuildThreads) {
            const int win = max(resp_off[i + 1] - resp_off[i], 0);
            np += min(max(keep_len[i], 0), win);
            nv += done[i] != 0 ? win : 0;
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        np += __shfl_down(np, off);
        nv += __shfl_down(nv, off);
    }
    if (lane == 0) {
        s.part[0][wave] = np;
        s.part[1][wave] = nv;
    }
    __syncthreads();
    if (tid == 0) {
        np = nv = 0;
        for (int w = 0; w < kBuildWaves; ++w) {
            np += s.part[0][w];
            nv += s.part[1][w];
        }
        pl.hdr->n_policy = np;
        pl.hdr->n_value = nv;
        pl.hdr->has_sets = keep_len ? 1 : 0;
    }
}

// Workgroup `g` of `groups` zeroes its share of the tagged words.
__device__ __forceinline__ void clear_words(const Plan& pl, int g, int groups) {
    typedef unsigned long long two __attribute__((ext_vector_type(2)));
    const int64_t pairs = plan_words(pl.cap) / 2;                   // (256-byte aligned, a whole number of 256 bytes)
    two* at = reinterpret_cast<two*>(pl.scan_words);
    for (int64_t i = (int64_t)g * kBuildThreads + threadIdx.x; i < pairs; i += (int64_t)groups * kBuildThreads)
        at[i] = two{0ull, 0ull};
}

}  // namespace tppo
