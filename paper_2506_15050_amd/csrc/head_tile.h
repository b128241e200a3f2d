// Machinery shared by the LM-head kernels: the XCD-aware sweep of MFMA tiles
// (W-role rows x token-role rows) with a pluggable per-lane epilogue, as 256 x 256
// tiles on a persistent grid or, where those leave the chip idle, with a workgroup
// per task, as 256 x 64, 128 or 192 tiles (narrow) or 128 x 64 ones (small).  K is
// contiguous in both operands, or the row index of one (KMAJOR).  The forward pass plugs in the online log-softmax; the backward
// pass plugs in the softmax-derivative writer and a plain tile store, which makes
// the sweep a matrix product.
#pragma once
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "common.h"

namespace tppo {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr int kMaxSplits = 256;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
// finite stand-ins for -inf (they keep exp2(m - m') NaN-free)
constexpr float kNegBig = -3.0e38f;    // in units of log2
constexpr float kLowest = -3.402823466e38f;   // in units of the logits: no finite one lies below

// A block of the sweep's work: `rows` token tiles from `row0` on, `cols` divisions of the W-role side each (see
// "Schedule" below).
struct Grid {
    int row0, rows, cols;
};

struct HeadParams {
    const void* hidden;
    const void* w;
    const int32_t* sel_rows;
    const int32_t* sel_targets;
    const int64_t* m_actual;
    int64_t n_rows, ld_h, ld_w, M;
    int H, V, row_tiles;
    int vocab_tiles, v_unit;           // what the columns of a grid divide: so many tiles (or parts of one) of v_unit rows
    int k_tiles;                       // K stages: H / kBK, rounded up
    // schedule
    Grid first, rest;                  // tasks 0 .. first_tasks - 1 come from `first`, the others from `rest`
    int first_tasks, rest_base, rest_tasks, k_chunks;
    int n_tasks;                       // first_tasks + rest_tasks * k_chunks
    int32_t* arrivals;                 // [256] the round each workgroup has come to; NULL: one round, nothing to align
    // partial results: of the log-softmax ([3][cols][tokens of the grid] per grid: max in the log2 domain, sumexp,
    // target logit), or of the tiles whose contraction is cut into k_chunks ([chunk][task][256 x 256])
    float *part_first, *part_rest;
    // used by the epilogues of the backward pass only
    const float* aux0;                     // per-token scalars (lse)
    const float* aux1;                     // per-token scalars (upstream derivative)
    const int32_t* aux_index;              // where token t's scalars sit in aux0/aux1 (NULL: at t)
    void* out;                             // tile output
    int64_t ld_out, out_cols;              // leading dimension / columns of `out` that exist
    int accumulate;                        // add to `out` instead of overwriting it
    int km_rows, km_cols;                  // a K-major operand: K rows that exist (zeros beyond), columns that exist
};

// The kernel's shape: a kTileV x kTileT (vocabulary x tokens) output tile per workgroup of kWavesV x kWavesT
// wavefronts, kBK K-elements per LDS stage, two stages.
//
// LDS staging layout.  A stage holds kTileV + kTileT rows of kBK bf16 (W rows
// first, then token rows), each row as kBK/8 chunks of 16 bytes.  Chunk c of
// row r sits in slot c ^ swz(r).  The LDS serves 64 banks x 4 B = 256 B per
// cycle, i.e. 16 lanes of a ds_read_b128; those 16 lanes read the same chunk
// of 16 consecutive rows, and the swizzle spreads them over all 16 slots of
// the 256-byte bank window (measured: SQ_LDS_BANK_CONFLICT = 0).
//
// The element type T is bf16 (uint16_t) or float; a stage's row is 128 bytes either way, and so are all transfers
// and fragments.  fp32 runs four v_mfma_f32_16x16x4_f32 on a pair of 16-byte fragments: MFMA j takes element j of
// every lane's chunk, i.e. k = j, 4 + j, 8 + j, 12 + j of the 16 -- the same set on both sides, in another order.
// Its matrix rate is a sixteenth of bf16's, so nothing else matters there (measured: 2064 tokens, H = 1024,
// V = 32000: 1.1 ms, 124 TFLOP/s of the 154 a large fp32 product reaches here; one token per workgroup with
// plain multiply-adds took 77-80 ms).
//
// For bf16 the MFMA is v_mfma_f32_16x16x32_bf16: same flops per cycle and same LDS bytes per flop as 32x32x16, but at the
// chip's power limit it sustains more (MFMA loop on LDS-fed fragments: 1.65 vs 1.55 PFLOP/s; on register-resident
// ones 2.10 vs 1.83).  Lane l of a wave holds, for a 16 x 16 block, column l % 16 (a token) and rows
// (l/16)*4 + e, e < 4 (vocabulary entries), and reads its operand fragments as 16 bytes: row l % 16, K chunk
// l / 16 of the MFMA's K range.
// RAGGED: H is not a multiple of a stage, and the chunks of the last one that lie beyond it are fetched as zeros (a
// variant of its own: the selects cost registers that the plain one does not have to spare).
// SMALL: 128 x 64 tiles and workgroups of 2 x 2 wavefronts, three to a CU, for calls that would leave much of the
// chip idle with the large ones (plan_small has the line between them).
// TOKEN_BLOCKS < 4 (bf16): narrow tiles, 256 x 64 TOKEN_BLOCKS, and a workgroup per task too: the large tile's workgroup and
// W rows, for calls of some tens to some hundreds of tokens (plan_narrow).
// FEW (small tiles): no more than two workgroups to a CU, whose stages' transfers go out early: spread over the whole stage the
// last ones are waited for in vain where no third workgroup computes meanwhile.  fp32, us, late -> early, one workgroup to a CU:
// 1600 tokens x V 32000, H 1024: 1184 -> 955;  4000 x 5000, H 2048: 939 -> 761;  two: 2064 x 45000, H 1024: 1647 -> 1604;  three: 2064 x
// 32000: 1101 (1109);  3300 x 32000: 1788 (1807).
// LONG (large tiles, the log-softmax over kLongStages and more): a task's set-up and its steps from tile to tile as they fit the K loop best.
// Elsewhere they are lean: the parameters asked for anew by every task instead of kept over all, spilled lane by lane (params_again), the
// rows of the token list all at once instead of one by one, a step to the next tile of W rows instead of every row's address.  us, LONG ->
// lean:  5000 tokens x V 30000, H 64: 51.1 -> 48.2;  20000 x 10000, H 128: 85.0 -> 80.5;  13640 x 32000, H 1024: 665 -> 657;  8000 x 40000, H 2048:
// 924 -> 918; narrow, 500 x 12000, H 1024: 27.4 -> 25.4;  900 x 5000, H 2048: 41.2 -> 39.2; ragged, 2516 x 50021, H 1000: 225.7 -> 222.9.  Where a
// set-up hardly counts, the loop that the compiler makes of the rest does, 8 bytes on from the other's place in a fetched line: 6000 x 50000,
// H 2560: 1184 -> 1187;  12000 x 32000, H 4096: 2302 -> 2311;  4000 x 50000, H 3584: 1085 -> 1091;  H 5120: 1551 -> 1564;  20000: 7277 -> 7330;  942 x
// 152064: 1252 -> 1261; though 6000 x 50000, H 2304: 1042 -> 1035;  8000 x 40000, H 3072: 1438 -> 1432.  The derivative's sweep is lean at any
// length: 1500 x 9001, H 1600: 47.4 -> 46.2;  8206 x 32000, H 1792: 794 -> 788;  H 2304: 993 -> 983;  H 3584: 1496 -> 1483;  8000 x 100000, H 4096:
// 4897 -> 4870;  3514 x 152064, H 5120: 4284 -> 4287;  9000: 10506 -> 10492;  40000 x 32000, H 2048: 4317 -> 4319.
// KMAJOR (bf16, large tiles): one operand lies in memory with K as the ROW index -- 1 the W-role one, 2 the token-role
// one; element (row r, k) is at base[k * ld + r].  A stage of it is kBK rows of 512 bytes, K row k's 16-byte chunk c in
// slot c ^ swz_k(k), and ds_read_b64_tr_b16 takes fragments out transposed: 16 lanes read 4 K rows x 16 columns, lane i
// gets column i's four.  Two of them make the fragment one ds_read_b128 gives of the other layout.
constexpr int kLongStages = 36;
template <typename T, bool RAGGED, bool SMALL = false, int KMAJOR = 0, int TOKEN_BLOCKS = 4, bool FEW = false, bool LONG = false>
struct HeadCfg {
    static constexpr bool kRagged = RAGGED, kSmall = SMALL, kLong = LONG;
    static constexpr int kKMajor = KMAJOR;
    static constexpr bool kOneTile = KMAJOR != 0;      // products: a task is one output tile
    static constexpr int kEsz = sizeof(T), kPerChunk = 16 / kEsz;         // elements of a 16-byte chunk
    typedef typename std::conditional<kEsz == 2, bf16x8, f32x4>::type Frag;
    static constexpr int kMI = 16, kGroups = 64 / kMI, kAccElems = 4;
    typedef float Acc __attribute__((__vector_size__(kAccElems * sizeof(float))));
    static constexpr bool kNarrow = TOKEN_BLOCKS != 4;
    static constexpr int kTileV = SMALL ? 128 : 256, kTileT = SMALL ? 64 : 64 * TOKEN_BLOCKS;
    static constexpr int kWavesV = 2, kWavesT = SMALL ? 2 : 4, kBK = 128 / kEsz, kStages = 2;
    static constexpr int kGroupsPerCu = SMALL ? 3 : 1;
    // The log-softmax's running maximum is held in logits in fp32, whose sweep the matrix cores bound: no finite logit is out
    // of its range.  In bf16 it is held in units of log2, rounded, one operation per logit less (ragged rows: 1 % at H = 1000,
    // 5 % at H = 72), and the merge takes that rounding back out (head.hip).
    static constexpr bool kLogitMax = sizeof(T) == 4;
    // Small tiles and narrow ones of up to 128 tokens have registers for a second set of accumulators: every kSumStages stages
    // (128 elements of K) what the matrix cores have added up moves there, so that no sum runs over thousands of elements one
    // after the other.
    static constexpr int kSumStages = SMALL || TOKEN_BLOCKS <= 2 ? 128 / kBK : 0;
    static constexpr int kWaves = kWavesV * kWavesT, kThreads = kWaves * 64;
    static constexpr int kWaveV = kTileV / kWavesV, kWaveT = kTileT / kWavesT;    // wave tile
    static constexpr int kVB = kWaveV / kMI, kTB = kWaveT / kMI;                  // 16 x 16 blocks per wave
    // an MFMA step: one W block over four chunks of K, against all token blocks
    static constexpr int kMfmaPerStep = kTB;
    static constexpr int kRowBytes = kBK * kEsz, kChunks = kRowBytes / 16;
    static constexpr int kRows = kTileV + kTileT;
    static constexpr int kStageBytes = kRows * kRowBytes;
    // W's lines are brought into L2 ahead of their transfers (head_mfma_kernel, prefetch)
    static constexpr bool kPrefetch = kEsz == 2 && !SMALL && (RAGGED || kNarrow);
    static constexpr int kLdsBytes = kStages * kStageBytes + (kEsz == 2 && !SMALL ? 256 : 0);
    static constexpr int kRowsPerDma = 1024 / kRowBytes;                  // one wave-wide 16 B/lane transfer
    static constexpr int kDmaPerStage = kRows / kRowsPerDma;
    static constexpr int kDmaPerWave = kDmaPerStage / kWaves;
    static constexpr int kKSteps = (kChunks / 4) * kVB;
    // a wave issues the transfers of a stage one by one between its next kSpread MFMAs, so that it never sits in
    // a full memory queue.  Small tiles, over 16 (all there are) / 14 / 12 / 10 / 8 of fp32's groups of four: 2064 tokens x V 32000, H 1024 1100 /
    // 1095 / 1089 / 1109 / 1109 us;  6000 x 32000 3168 / 3144 / 3127 / 3183 / -;  2064 x 32000, H 256 290 / 290 / 289 / 294 / -: three workgroups cover
    // for each other, but not for transfers that go out at a stage's end and are waited for there.  (Without transfers, 1024 us.)  bf16, over all
    // 16 MFMAs -> 12: log-probs, 146 x V 5000, H 1024 15.1 -> 14.5;  700 x 6000, H 256 14.4 -> 14.0;  300 x 1000, H 256 9.10 -> 8.98;  1030 x 3000,
    // H 64 9.26 -> 9.25; backward calls 0 to 1 % (146 x 5000 56.5 -> 55.8, 358 x 11732, H 192 58.9 -> 58.7); none of twelve sizes slower.
    static constexpr int kSpread = FEW ? 8 : SMALL ? 12 : TOKEN_BLOCKS == 1 ? 16 : 8 * TOKEN_BLOCKS;
    static_assert(kDmaPerWave * kWaves == kDmaPerStage, "transfers must divide evenly over the waves");
    static_assert(kTileV % kRowsPerDma == 0, "a transfer may not straddle W and token rows");
    static_assert(kKSteps % 2 == 0, "fragment double buffering assumes an even number of K steps");
    static_assert(kWavesV * 3 * kTileT * 4 <= kLdsBytes, "merge buffer must fit in the idle stages");
    static_assert(kStages == 2 && kSpread <= kKSteps * kMfmaPerStep, "spread issue: at most one stage's worth of MFMAs");
    __device__ static __forceinline__ int swz(int r) { return (r >> 1) & 7; }
    __device__ static __forceinline__ int chunk_off(int r, int c) { return r * kRowBytes + ((c ^ swz(r)) << 4); }
    // K-major operand: the 32 lanes that a tr read serves at a time cover 8 K rows, {0 .. 3, 8 .. 11} + 4 h (mod 16),
    // of 32 bytes each; this spreads them over the 8 places of the 256-byte bank window
    static constexpr int kKRowBytes = 512;
    __device__ static __forceinline__ int swz_k(int k) { return ((k & 3) | ((k >> 3) & 1) << 2) << 1; }
    static_assert(KMAJOR == 0 || (kEsz == 2 && !SMALL && !RAGGED && kTileV * kEsz == kKRowBytes && kTileT == kTileV),
                  "K-major stages are laid out for 256 columns of 2 bytes");
    // dZ lies in blocks of 64 rows x 64 columns, 8 KB each, a row of blocks after the other: a stage of the first product (256
    // rows x 64 of K) is four blocks, one of the second (64 of K x 256 columns) four that follow each other, and both walk on
    // by whole blocks, where rows of V entries gave 128 or 512 bytes of each of 256 or 64 rows.  First product, dZ row by row ->
    // in blocks, us: 16414 tokens x V 32000, H 1024: 889 -> 854;  3514 x 152064, H 5120: 4251 -> 4220; the second and the stores: the same.
    // Byte of element (r, c), `cols` columns in all, a multiple of 64:
    static constexpr int kBlockBytes = 64 * 64 * 2;
    __device__ static __forceinline__ int64_t block_at(int64_t r, int64_t c, int64_t cols) {
        return ((r >> 6) * (cols >> 6) + (c >> 6)) * kBlockBytes + (r & 63) * 128 + (c & 63) * 2;
    }
    // row (inside the wave tile's W rows) of accumulator element e of block vb, for lane group g = lane / 16
    __device__ static __forceinline__ int row_in_wave(int vb, int e, int g) { return vb * kMI + g * 4 + e; }
};

// One wave-wide global -> LDS transfer without a register round trip: lane l's
// 16 bytes at `src` land at LDS byte address lds_base + 16*l (lds_base is
// wave-uniform and goes through M0; `lds_offset` is a constant that is added; the
// transfer may not follow the write of M0 at once).  Written as inline assembly so
// that the transfer stays asynchronous: completion is awaited by hand (vmcnt) right
// before the workgroup barrier that publishes the stage.
__device__ __forceinline__ void dma_16b_per_lane(const void* src, unsigned lds_base, int lds_offset) {
    asm volatile("s_add_u32 m0, %0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 :
                 : "s"(lds_base), "v"(src), "i"(lds_offset)
                 : "memory", "m0", "scc");
}

// The same with 4 bytes a lane, 256 bytes in all.
__device__ __forceinline__ void dma_4b_per_lane(const void* src, unsigned lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off"
                 :
                 : "s"(lds_base), "v"(src)
                 : "memory", "m0");
}

// s_waitcnt immediate that waits for vmcnt <= n only (gfx9 encoding)
constexpr int vmcnt_imm(int n) { return (n & 0xF) | ((n >> 4) << 14) | (0x7 << 4) | (0xF << 8); }

constexpr int kLgkm0 = 0xF | (3 << 14) | (0x7 << 4);      // ... and one that waits for LDS reads only

// Schedule.  The launch of the large tiles is persistent: 256 workgroups, one per CU; hardware id b runs on XCD b % 8 (ids go
// round-robin over the 8 XCDs, each with its own L2).  The work is a list of tasks, 256 to a round, dealt out so
// that the 32 workgroups of an XCD hold 32 CONSECUTIVE tasks.  A grid of `rows` token tiles x `cols` divisions of
// the W-role side is listed in blocks of 8 rows, column by column: an XCD's 32 tasks are 8 token tiles x 4
// columns, so every W tile is wanted by 8 of its workgroups and every token tile by 4 at the same step of equal
// sweeps; one of them pays the L2 miss and the others hit (ideal hit rate 1 - 12/64 = 81 %, 80.9 % measured).
// (A free-running grid drifts apart and reached 51-58 %.)  Across XCDs a round covers consecutive blocks, so the
// XCDs sweep the same W rows at about the same time and W leaves HBM once per round.
//
// The list has two parts (host side: plan_sweep / plan_product): whole rounds of the division that shares best,
// and the rest, which is fewer token tiles (or output tiles) than fill a round and is cut finer, so that no
// workgroup idles through a last round.
//   log-softmax and dz sweeps:  a column is a range of vocabulary tiles; `rest` is the last token tiles, with
//                               more vocabulary splits.
//   plain products:             a column is one tile of W-role rows; `rest` is the last output tiles, each cut
//                               into k_chunks of the contraction, whose partial tiles a second kernel adds up.
// Workgroups of an XCD re-align at every round boundary.  That wait is only a hint for
// the caches: it is bounded and falls through, and nothing depends on it.  Plain products of up to kAlignStages stages go without:
// their workgroups would store 64 MB of output tiles all at the same time, and a contraction of some stages is short against that.
// Over thousands of stages those that drift apart read from HBM what their neighbours had in L2.  Waiting for each other -> not, us:
//   stages      2: V 46863 x H 3520, 185 tokens: d/dW 205 -> 170        26: 54342 x 1664, 1722: d/dW 328 -> 319
//              54: 152064 x 5120, 3514: d/dW 4536 -> 4459              125: 152064 x 5120, 8000: d/dW 9403 -> 9422
//             256: 32000 x 1024, 16414: d/dW 870 -> 852                312: 152064 x 5120, 20000: d/dW 23372 -> 23306
//             500: 32000 x 4096, 20000: d/dh 3854 -> 3830; 40000: 7804 -> 7887; 32000 x 1024, 16414: 828 -> 818
//             625: 64000 x 2048, 40000: d/dW 7992 -> 8015             1000: 64000 x 5120, 30000: d/dh 14703 -> 14924
//            1211: 152064 x 5120, 77528: d/dW 88920 -> 89951           937: 16000 x 4096, 60000: d/dW 5910 -> 5922
//            2376: 152064 x 5120, 20000: d/dh 23414 -> 23749; 77528: 91866 -> 95332 (another card: 92100 -> 100500)
// Small and narrow tiles have one list (`rest`), a workgroup per task up to 2^20 of them, and no re-alignment.
constexpr int kSweepGroups = 256, kXcdGroups = kSweepGroups / 8, kRowBlock = 8;
constexpr int kAlignSpins = 4096, kAlignStages = 512;
// Every workgroup says in a word of its own which round it has come to (0 when it starts) and waits for the words of its
// XCD's workgroups that have a task in that round.  Nothing has to be cleared before the launch, as counters had to be: 20000 tokens
// x V 4000, H 320: 84 -> 76 us; 13640 x 32000, H 1024: 4.6 us of a launch less.  Without any re-alignment H = 5120 loses 8 % on 63263
// tokens x V 152064 (1.7 times the misses in L2), H = 3584 1 %.
__device__ __forceinline__ void arrive(int32_t* rounds, int xcd, int slot, int round) {
    if (threadIdx.x == 0) __hip_atomic_store(rounds + xcd * kXcdGroups + slot, round, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void align_round(int32_t* rounds, int xcd, int slot, int round, int expected) {
    arrive(rounds, xcd, slot, round);
    if (threadIdx.x < kWave) {
        const int other = min((int)threadIdx.x, expected - 1);
        for (int spin = 0; spin < kAlignSpins; ++spin) {
            const int at = __hip_atomic_load(rounds + xcd * kXcdGroups + other, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (__all(at >= round)) break;
            __builtin_amdgcn_s_sleep(8);
        }
    }
    __syncthreads();
}

struct Task {
    int row, col;                      // token tile, column of its grid
    int v_begin, v_end;                // W-role rows; tiles of kTileV from v_begin on
    int k_begin, k_tiles;              // K range in steps of kBK
    int rest;                          // which grid: 0 first, 1 rest
    int part;                          // rest: index of the partial tile (chunk * rest_tasks + task)
};

template <bool ONE_TILE>
__host__ __device__ __forceinline__ Task task_at(const HeadParams& p, int t, int all_k_tiles) {
    Task x;
    x.rest = t >= p.first_tasks;
    Grid g = p.first;
    int id = t, chunk = 0;
    x.part = 0;
    x.k_begin = 0;
    x.k_tiles = all_k_tiles;
    if (x.rest) {
        g = p.rest;
        x.part = t - p.first_tasks;
        id = p.rest_base + x.part;
        if (p.k_chunks > 1) {
            chunk = x.part / p.rest_tasks;
            id -= chunk * p.rest_tasks;
            x.k_begin = (int)((int64_t)all_k_tiles * chunk / p.k_chunks);
            x.k_tiles = (int)((int64_t)all_k_tiles * (chunk + 1) / p.k_chunks) - x.k_begin;
        }
    }
    const int block = id / (kRowBlock * g.cols), in_block = id - block * (kRowBlock * g.cols);
    const int height = min(kRowBlock, g.rows - block * kRowBlock);
    x.col = in_block / height;
    x.row = g.row0 + block * kRowBlock + in_block - x.col * height;
    // Products, whose column is a tile, divide nothing more.  Backward calls, us, with the columns' division, twice per task -> without:
    // 64 tokens x V 2000, H 64: 25.6 -> 25.2;  225 x 11194, H 2304: 106.8 -> 105.9;  61 x 54900, H 1728: 190.8 -> 189.8;  185 x 46863, H 3520: 407 -> 405.
    if (ONE_TILE) {
        x.v_begin = x.col * p.v_unit;
        x.v_end = min(p.V, x.v_begin + p.v_unit);
        return x;
    }
    // vocab_tiles * col / cols and the same of col + 1, without 64-bit divisions: quotient and remainder of vocab_tiles by cols
    const unsigned cols = g.cols, each = (unsigned)p.vocab_tiles / cols, over = (unsigned)p.vocab_tiles - each * cols;
    const unsigned begin = over * x.col / cols, end = begin + (over * x.col - begin * cols + over >= cols);
    x.v_begin = (int)(each * x.col + begin) * p.v_unit;
    x.v_end = (int)min((int64_t)p.V, (int64_t)(each * (x.col + 1) + end) * p.v_unit);
    return x;
}

// The kernel's parameters where the launch left them, asked for anew: `HeadParams` has more words than there are scalar registers to keep
// them in over the tasks, and what is kept is spilled lane by lane and read back at every use.
__device__ __forceinline__ const HeadParams& params_again(const HeadParams& p) {
#ifdef __HIP_DEVICE_COMPILE__
    typedef const HeadParams __attribute__((address_space(4))) * Args;
    Args at = (Args)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(at));
    return *(const HeadParams*)at;
#else
    return p;
#endif
}

// Epi (the per-lane epilogue) provides
//   init(p, tok0, m_eff, wt, lane)                          once per task,
//   fold(acc, p, task, tok0, m_eff, v0, wv, wt, lane)       after each finished tile of W rows; clears acc,
//   finish(p, lds_scratch, task, tok0, m_eff, wv, wt, lane, tid)  after the task's tiles (workgroup-wide),
//   kPrefetch  W's lines brought ahead in large tiles,   kDealt  small tiles dealt out one by one (launch_sweep).
// what the chunks beyond a ragged H hold, in both operands
static __device__ const uint4 kZeroChunk = {0, 0, 0, 0};

template <class C, template <class> class Epi>
__global__ __launch_bounds__(C::kThreads, C::kGroupsPerCu * C::kWaves / 4) void head_mfma_kernel(HeadParams args) {
    constexpr int kTileV = C::kTileV, kTileT = C::kTileT, kWaveV = C::kWaveV, kWaveT = C::kWaveT;
    constexpr int kVB = C::kVB, kTB = C::kTB;
    constexpr int kDmaPerWave = C::kDmaPerWave, kKSteps = C::kKSteps;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int64_t m_eff = args.m_actual ? min(args.M, *args.m_actual) : args.M;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wv = wave / C::kWavesT, wt = wave % C::kWavesT;
    const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;

    constexpr bool kPersistent = !C::kSmall && !C::kNarrow;
    if (kPersistent && args.arrivals) arrive(args.arrivals, xcd, slot, 0);
    const bool dealt = C::kSmall && Epi<C>::kDealt && args.rest.rows > 1;
    const int t_first = dealt ? (int)blockIdx.x : xcd * ((int)gridDim.x >> 3) + slot, t_step = (int)gridDim.x;
    for (int t = t_first, n_tasks = args.n_tasks; t < n_tasks; t += t_step) {
    const HeadParams& p = C::kLong ? args : params_again(args);
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                           // a task's own: nothing derived from it is kept over the others
    const int lane = tid & 63, frag_row = lane % C::kMI, frag_grp = lane / C::kMI;
    const int round = t / kSweepGroups;
    if (kPersistent && round > 0 && p.arrivals)            // the first round starts aligned
        align_round(p.arrivals, xcd, slot, round, min(kXcdGroups, p.n_tasks - (t - slot)));
    const Task task = task_at<C::kOneTile>(p, t, p.k_tiles);
    const int64_t tok0 = (int64_t)task.row * kTileT;
    if (tok0 >= m_eff) continue;                            // uniform over the workgroup
    const int v_end = task.v_end, k_tiles = task.k_tiles;
    const int total_iters = (v_end - task.v_begin + kTileV - 1) / kTileV * k_tiles;

    // ---- loader role: transfers wave*kDmaPerWave + q, each kRowsPerDma staged rows
    const int ld_row0 = wave * kDmaPerWave * C::kRowsPerDma + lane / C::kChunks;   // + q * kRowsPerDma
    const int ld_slot = lane % C::kChunks;
    const char* src[kDmaPerWave];
    const int k_bytes = p.H * C::kEsz;
    const int64_t ld_w = p.ld_w * C::kEsz, ld_h = p.ld_h * C::kEsz;
    // this wavefront's transfers are all of one operand
    constexpr int kVWaves = C::kKMajor ? kTileV / (kDmaPerWave * C::kRowsPerDma) : 1;
    const bool k_major = (C::kKMajor == 1 && wave < kVWaves) || (C::kKMajor == 2 && wave >= kVWaves);
    const int km_row0 = (wave & (kVWaves - 1)) * kDmaPerWave * 2 + (lane >> 5);          // + q * 2: K row in the stage
    // (64 bits throughout: a transfer adds its stage's offset to an address, and 32 are extended every time.  Calls, us, 32 -> 64:
    // 6254 tokens x V 1373, H 64: 18.8 -> 17.9;  177 x 44067, H 128: 22.2 -> 21.3;  942 x 152064, H 5120: 1289 -> 1281.)
    const int64_t k_step = k_major                            ? C::kBK * (C::kKMajor == 1 ? ld_w : ld_h)
                           : C::kKMajor == 1 && wave >= kVWaves ? C::kBlockBytes
                                                                : C::kRowBytes;
    const int64_t k_first = task.k_begin * k_step;
    int issue_v = task.v_begin, issue_kt = 0;
    // Where this wavefront's transfers land, in one stage and the other in turn: one scalar register, and one scalar instruction a
    // transfer.  (A place for each transfer held eight, some of them spilled and read back by every stage: 63263 tokens x
    // V 152064, H 5120: 70.3 -> 68.7 ms;  942 x 152064: 1313 -> 1279 us;  16000 x 32000, H 1024: 829 -> 806;  2516 x 50021, H 1000:
    // 242 -> 240;  fp32, 2064 x 32000, H 1024: 1113 -> 1106.)
    const unsigned dst_first = lds_base + wave * kDmaPerWave * 1024;
    unsigned issue_dst = dst_first;
    int64_t issue_kpos = k_first;
    int issue_left = p.km_rows - task.k_begin * C::kBK;                 // K rows from the stage to be issued on
    auto token_of = [&](int q) {
        const int64_t t = min(tok0 + (ld_row0 + q * C::kRowsPerDma - kTileV), m_eff - 1);
        return t < 0 ? (int64_t)0 : t;                                 // (a W row's)
    };
    constexpr int kRowsPerWave = kDmaPerWave * C::kRowsPerDma;
    auto is_w_row = [&](int q) {                                       // (the same for all lanes)
        return !C::kLong && kTileV % kRowsPerWave == 0 ? wave < kTileV / kRowsPerWave : (wave * kDmaPerWave + q) * C::kRowsPerDma < kTileV;
    };
    auto point_at_tile = [&](int v0, bool w_only) {
        // The token rows that this wavefront stages, all of them asked for at once: one by one each is waited for before the next
        // transfer's, eight trips to memory.
        int listed[kDmaPerWave];
        if (!C::kLong && C::kKMajor == 0 && p.sel_rows && !is_w_row(kDmaPerWave - 1)) {
#pragma unroll
            for (int q = 0; q < kDmaPerWave; ++q) listed[q] = p.sel_rows[token_of(q)];
        }
#pragma unroll
        for (int q = 0; q < kDmaPerWave; ++q) {
            if (C::kKMajor && k_major) {                                // (columns that do not exist: any others, never stored)
                const int k = km_row0 + 2 * q, col = ((lane & 31) ^ C::swz_k(k)) * 8;
                if (C::kKMajor == 1)
                    src[q] = static_cast<const char*>(p.w) + k * ld_w + (int64_t)min(v0 + col, p.km_cols - 8) * C::kEsz;
                else
                    src[q] = static_cast<const char*>(p.hidden) +
                             C::block_at(k, min(tok0 + col, (int64_t)p.km_cols - 8), p.ld_h);
                continue;
            }
            const int r = ld_row0 + q * C::kRowsPerDma;                 // staged row; < kTileV means a W row
            const int chunk = (ld_slot ^ C::swz(r)) * 16;
            if (is_w_row(q)) {
                const int64_t v = min(v0 + r, v_end - 1);
                src[q] = static_cast<const char*>(p.w) + v * ld_w + chunk;
            } else if (!w_only) {
                const int64_t t = C::kLong ? min(tok0 + (r - kTileV), m_eff - 1) : token_of(q);
                if (C::kKMajor == 1) {
                    src[q] = static_cast<const char*>(p.hidden) + C::block_at(t, 0, p.ld_h) + chunk;
                    continue;
                }
                int64_t row = p.sel_rows ? (int64_t)(C::kLong ? p.sel_rows[t] : listed[q]) : t;      // no list: rows in order
                row = min(max(row, (int64_t)0), p.n_rows - 1);
                src[q] = static_cast<const char*>(p.hidden) + row * ld_h + chunk;
            }
        }
    };
    // On to the next tile of W rows, the one from v0 on: the same step for all rows, but in a last tile with fewer of them, where what lies
    // beyond is the last row again.  (Each row's address from its number takes three multiplications of 16 cycles.)
    const int64_t w_step = (int64_t)kTileV * ld_w;
    auto next_w_tile = [&](int v0) {
        if (!is_w_row(0)) return;
        if (v0 + kTileV <= v_end) {
#pragma unroll
            for (int q = 0; q < kDmaPerWave; ++q)
                if (is_w_row(q)) src[q] += w_step;
        } else {
#pragma unroll
            for (int q = 0; q < kDmaPerWave; ++q)
                if (is_w_row(q)) src[q] += min(kTileV, v_end - 1 - v0 - (ld_row0 + q * C::kRowsPerDma) + kTileV) * ld_w;
        }
    };
    auto point_at_zeros = [&]() {       // a K-major operand's rows beyond the last K row, in a tile's last stage
        if (C::kKMajor && k_major && issue_left < C::kBK) {
#pragma unroll
            for (int q = 0; q < kDmaPerWave; ++q)
                if (km_row0 + 2 * q >= issue_left) src[q] = reinterpret_cast<const char*>(&kZeroChunk) - issue_kpos;
        }
    };
    point_at_tile(task.v_begin, false);
    point_at_zeros();
    // Ragged rows: the lanes whose chunk of a tile's last stage lies beyond H, the same ones in every other transfer, take zeros
    // for it.  `zeros`: those lanes if the stage to be issued is a last one.  Masks and two selects a transfer; a branch for the last
    // stage at every one of them took, us: 2516 tokens x V 50021, H 1000: 260 (now 245);  4000 x 9000, H 520: 60.6 (57);  900 x 12000,
    // H 2040: 79.4 (77.5);  12000 x 9000, H 136: 78.7 (75.1);  300 x 20000, H 72: 20.8 (20.2).
    const int last_kpos = (p.k_tiles - 1) * C::kRowBytes;
    uint64_t beyond[2] = {}, zeros[2] = {};
    const char* zero_chunk = reinterpret_cast<const char*>(&kZeroChunk);
    auto find_zeros = [&]() {
        if constexpr (C::kRagged) {
#pragma unroll
            for (int i = 0; i < 2; ++i) zeros[i] = issue_kpos == last_kpos ? beyond[i] : 0;
        }
    };
    if constexpr (C::kRagged) {
        asm volatile("" : "+v"(zero_chunk));
#pragma unroll
        for (int i = 0; i < 2; ++i) beyond[i] = __ballot(last_kpos + (ld_slot ^ C::swz(ld_row0 + i * C::kRowsPerDma)) * 16 >= k_bytes);
        find_zeros();
    }
    auto issue_one = [&](int q) {
        const char* from = src[q] + issue_kpos;
        if (C::kRagged) from = __builtin_amdgcn_inverse_ballot_w64(zeros[q & 1]) ? zero_chunk : from;
        dma_16b_per_lane(from, issue_dst, q * 1024);
    };
    auto issue_advance = [&]() {        // next (vocabulary tile, k tile) in sweep order
        issue_kpos += k_step;
        issue_left -= C::kBK;
        issue_dst = 2 * dst_first + C::kStageBytes - issue_dst;
        if (!C::kOneTile && ++issue_kt == k_tiles) {
            issue_kt = 0;
            issue_kpos = k_first;
            issue_v += kTileV;
            if (C::kLong) point_at_tile(issue_v, true);
            else next_w_tile(issue_v);
        }
        point_at_zeros();
        find_zeros();
    };
    // ---- Prefetch.  A stage's transfers go out in the first half of the stage before and are waited for at its end: time
    // enough for what lies in L2, hardly for a miss.  So kAhead stages before its transfers the 256 rows' lines of a stage of W
    // are touched, 64 by each of four wavefronts, with a transfer of 4 bytes a lane into a corner of LDS that nobody reads (a
    // load would hold registers until it returns).  Where workgroups of the XCD share the W tile (their token tiles
    // follow each other), each touches its part.  It is the last transfer that a wavefront has under way at a barrier, so
    // it is the one that may still be: the counter counts in order.
    // Measured with W in HBM, us a call: 2516 tokens x V 50021, H 1000: 270 -> 247;  300 x V 152064, H 5120: 604 -> 555;
    // 900 x V 20001, H 576: 38.0 -> 34.4;  100 x V 20000, H 4096: 87.1 -> 65.8;  20 x V 152064, H 5120: 352 -> 343.  Where W is in a
    // cache it costs: in calls one after the other on the same W 2 .. 3 % of ragged sweeps in large tiles (2516 x V 50021, H 1000:
    // 234 -> 240) and up to 10 % of narrow ones (1300 x V 12000, H 1024: 45.5 -> 50.0), and with W in HBM where all of it
    // stays in L2 from its first token tile on (8000 x V 1500, H 1000: 35.0 -> 36.5) or a row is two stages long (300 x V 20000, H 72:
    // 17.6 -> 19.1).  It stays on all the same: a pass over other tensors between two calls, as in a training step, leaves
    // little of W in a cache, and no call tells.  The touches add 5 % to the requests to L2 where four token tiles share them and
    // 39 % where one has them all, and none to the misses.
    // One stage ahead takes 271 us for the first, four 608 for the second.  Whole stages in large tiles lose by it (H = 3584:
    // 6 %, 1024: 3 %): all token tiles sweep the same W there, which is in a cache as it is, and the requests are a quarter
    // more.  Unless the epilogue's stores drive W out of L2 (DzAheadEpilogue).
    constexpr int kAhead = 2;
    constexpr bool kPrefetch = C::kPrefetch || Epi<C>::kPrefetch;
    const Grid& grid = task.rest ? p.rest : p.first;
    const bool prefetches = kPrefetch && wave >= 4 &&
                            ((wave ^ (task.row - grid.row0)) & (grid.rows >= 4 ? 3 : grid.rows >= 2 ? 1 : 0)) == 0;
    const char* ahead = nullptr;
    int ahead_v = task.v_begin, ahead_kt = 0;
    auto point_ahead = [&]() {
        ahead = static_cast<const char*>(p.w) + min(ahead_v + (wave & 3) * 64 + lane, v_end - 1) * ld_w;
    };
    auto prefetch_advance = [&]() {
        ahead += C::kRowBytes;
        if (++ahead_kt == k_tiles) {
            ahead_kt = 0;
            ahead_v += kTileV;
            point_ahead();
        }
    };
    auto prefetch = [&]() {
        if (kPrefetch && prefetches) {
            dma_4b_per_lane(ahead, lds_base + C::kStages * C::kStageBytes);
            prefetch_advance();
        }
    };
    auto wait_for_stage = [&]() {
        if (kPrefetch && prefetches) __builtin_amdgcn_s_waitcnt(vmcnt_imm(1));
        else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    };
    if (kPrefetch && prefetches) {
        point_ahead();
        for (int i = 0; i < 1 + kAhead; ++i) prefetch_advance();
    }
    Epi<C> epi;
    epi.init(p, tok0, m_eff, wt, lane);

    typename C::Acc acc[kVB][kTB];
#pragma unroll
    for (int vb = 0; vb < kVB; ++vb)
#pragma unroll
        for (int tb = 0; tb < kTB; ++tb)
#pragma unroll
            for (int e = 0; e < C::kAccElems; ++e) acc[vb][tb][e] = 0.f;

    // Fragments of MFMA step `step` of a stage (kKSteps steps per stage), double buffered: step = (four chunks of K) *
    // kVB + W block; the W block's fragment, K chunks 4 * (step / kVB) + group, and with a K step's first block
    // the token fragments of that K step.
    typename C::Frag fa[2], fb[2][kTB];
    // the fragment of 16 columns `block` of a K-major operand whose stage begins at LDS byte `at`; first_block: the
    // wave tile's (its column blocks are the 32-byte pieces first_block ... of a K row, exchanged by the swizzle)
    auto k_major_frag = [&](int at, int first_block, int block, int k32) {
        typedef short s4 __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) s4* lds_s4;
        const int k = frag_grp * 8 + (frag_row >> 2);                   // + 32 k32 + 4 h: neither changes the swizzle
        const int lane_at = k * C::kKRowBytes + ((2 * first_block + ((frag_row & 3) >> 1)) ^ C::swz_k(k)) * 16 + (frag_row & 1) * 8;
        const unsigned from = lds_base + at + (lane_at ^ (block * 32)) + k32 * 32 * C::kKRowBytes;
        const s4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(size_t)from);
        const s4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(size_t)(from + 4 * C::kKRowBytes));
        return __builtin_bit_cast(typename C::Frag, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto load_frags = [&](int stage, int step) {
        const unsigned char* st = smem + stage * C::kStageBytes;
        const unsigned char* a_base = st + (wv * kWaveV) * C::kRowBytes;
        const unsigned char* b_base = st + (kTileV + wt * kWaveT) * C::kRowBytes;
        const int k32 = step / kVB, vb = step % kVB, c = k32 * 4 + frag_grp;
        if constexpr (C::kKMajor == 1)
            fa[step & 1] = k_major_frag(stage * C::kStageBytes, wv * kVB, vb, k32);
        else
            fa[step & 1] = *reinterpret_cast<const typename C::Frag*>(a_base + C::chunk_off(vb * 16 + frag_row, c));
        if (vb == 0) {
#pragma unroll
            for (int tb = 0; tb < kTB; ++tb)
                if constexpr (C::kKMajor == 2)
                    fb[k32][tb] = k_major_frag(stage * C::kStageBytes + kTileV * C::kRowBytes, wt * kTB, tb, k32);
                else
                    fb[k32][tb] = *reinterpret_cast<const typename C::Frag*>(b_base + C::chunk_off(tb * 16 + frag_row, c));
        }
    };
    // An MFMA step with this wave's transfers of the stage being refilled issued between the MFMAs (`on` is
    // workgroup-uniform): transfer j follows MFMA number j * kSpread / kDmaPerWave, counted from the barrier that
    // freed the stage (`part`: steps since then).
    // The scheduling barrier in front keeps the next step's fragment reads ahead of this step's MFMAs; without it the
    // compiler puts each read right before its use, and half of the steps wait out the LDS latency (1 to 3 % of the
    // sweep, by card: the clock gives back part of what the shorter schedule gains).
    constexpr int kMfmaPerStep = C::kMfmaPerStep, kSpreadSteps = C::kSpread / kMfmaPerStep;
    auto mfma_step = [&](int step, int part, bool on) {
        const int k32 = step / kVB, vb = step % kVB;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int tb = 0; tb < kTB; ++tb) {
            if constexpr (C::kEsz == 2) {
                acc[vb][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[step & 1], fb[k32][tb], acc[vb][tb], 0, 0, 0);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[vb][tb] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[step & 1][j], fb[k32][tb][j], acc[vb][tb], 0, 0, 0);
            }
            if (part < kSpreadSteps) {
                if (on) {
#pragma unroll
                    for (int j = 0; j < kDmaPerWave; ++j)
                        if (j * C::kSpread / kDmaPerWave == part * kMfmaPerStep + tb) issue_one(j);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    // ---- fill the first stage, publish it, start on its first fragments
#pragma unroll
    for (int q = 0; q < kDmaPerWave; ++q) issue_one(q);
    issue_advance();
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __syncthreads();
    if (total_iters > 1) {
#pragma unroll
        for (int q = 0; q < kDmaPerWave; ++q) issue_one(q);
        issue_advance();
        prefetch();
    }
    load_frags(0, 0);

    typename C::Acc sums[C::kSumStages ? kVB : 1][C::kSumStages ? kTB : 1] = {};
    int kt = 0, v0 = task.v_begin, stage = 0;
    bool refill = false;                // transfers of the stage freed at the last barrier are pending
    for (int it = 0; it < total_iters; ++it) {
#pragma unroll
        for (int ks = 0; ks + 1 < kKSteps; ++ks) {
            load_frags(stage, ks + 1);
            mfma_step(ks, ks + 1, refill);
            if (ks + 2 == kSpreadSteps && refill) {
                issue_advance();
                prefetch();
            }
        }
        // The stage's last fragments are in registers.  Hand the stage back,
        // publish the next one and fetch its first fragments BEFORE issuing the
        // last MFMAs, so the barrier and the LDS latency hide behind them.
        refill = false;
        __builtin_amdgcn_s_waitcnt(kLgkm0);     // here, on both paths: behind the branch it would wait for the next stage's too
        if (it + 1 < total_iters) {
            wait_for_stage();
            __syncthreads();            // stage it+1 landed for everyone; everyone left stage it
            refill = it + 2 < total_iters;
            load_frags(stage ^ 1, 0);
        }
        mfma_step(kKSteps - 1, 0, refill);
        stage ^= 1;
        if (!C::kOneTile) ++kt;
        if constexpr (C::kSumStages != 0) {
            if (kt % C::kSumStages == 0 || kt == k_tiles) {
#pragma unroll
                for (int vb = 0; vb < kVB; ++vb)
#pragma unroll
                    for (int tb = 0; tb < kTB; ++tb) {
                        sums[vb][tb] += acc[vb][tb];
                        acc[vb][tb] = typename C::Acc{};
                    }
            }
        }
        if (!C::kOneTile && kt == k_tiles) {            // a tile is complete
            if constexpr (C::kSumStages != 0) epi.fold(sums, p, task, tok0, m_eff, v0, wv, wt, lane);
            else epi.fold(acc, p, task, tok0, m_eff, v0, wv, wt, lane);
            kt = 0;
            v0 += kTileV;
        }
    }
    if (C::kOneTile) epi.fold(acc, p, task, tok0, m_eff, v0, wv, wt, lane);
    if (kPrefetch) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));            // (this workgroup's LDS is somebody else's after its end)
    __syncthreads();                    // every fragment read is done before the stages are reused
    epi.finish(C::kLong ? args : params_again(args), reinterpret_cast<float*>(smem), task, tok0, m_eff, wv, wt, lane, tid);
    __syncthreads();                    // merge buffer is read before the next task's transfers land
    }
}

// ---- host side of the schedule
constexpr int kTile = 256;                         // both sides of an output tile

// What a task costs besides its tiles, in tile times of an H-deep sweep (pipeline fill, the wait at the round
// boundary, the merge at the end): 0.25 measured.
constexpr double kTaskCost = 0.25;
// The finer grid of the last token tiles stays within this many tasks, which bounds the partial results.
constexpr int64_t kRestTasks = 1024;

static double rounds_of(int64_t tasks) { return (double)((tasks + kSweepGroups - 1) / kSweepGroups); }

// Sweep of M token-role rows over V W-role rows, columns = ranges of W-role tiles.  Whole rounds take 64 token
// tiles x 4 columns (8 x 4 per XCD, the division with the least traffic; fewer columns when there are fewer W
// tiles); the token tiles that remain (or those and the last whole round's) get the number of columns that
// costs least.  Measured against equal units of 8 token tiles x 4 splits for everything, the last group of 8
// rounded up: 4 token tiles x 594 W tiles (10 instead of 19 tile times per workgroup; half of each unit's workgroups
// had no token tile) 2.24 -> 1.25 ms; 54 x 125 tiles 0.79 -> 0.75 ms; 227 x 594 tiles (533 instead of 574 tile
// times) 48.0 -> 45.6 ms; 248 x 594 (580 instead of 612) 1.3 %: there the busier chip clocks lower.
// Returns the cost.
static double plan_sweep(HeadParams& p, int64_t M, int64_t V) {
    p.M = M;
    p.V = (int)V;
    p.row_tiles = (int)((M + kTile - 1) / kTile);
    p.vocab_tiles = (int)((V + kTile - 1) / kTile);
    p.v_unit = kTile;
    const int rows = p.row_tiles, vts = p.vocab_tiles;
    int first_cols = vts < 4 ? (vts == 3 ? 2 : vts) : 4;            // 1, 2 or 4: a whole number of token tiles per round
    const int per_round = kSweepGroups / first_cols, most = rows / per_round;
    double best = 1e300;
    int best_rounds = 0, best_cols = 1;
    for (int k = most; k >= 0 && k + 1 >= most; --k) {
        const int64_t rest = rows - (int64_t)k * per_round;
        const double done = k * ((double)((vts + first_cols - 1) / first_cols) + kTaskCost);
        if (rest == 0) {
            if (done < best) { best = done; best_rounds = k; best_cols = 1; }
            continue;
        }
        for (int s = 1; s <= vts && s <= kMaxSplits && (s == 1 || rest * s <= kRestTasks); ++s) {
            const double cost = done + rounds_of(rest * s) * ((double)((vts + s - 1) / s) + kTaskCost);
            if (cost < best - 1e-9) { best = cost; best_rounds = k; best_cols = s; }
        }
    }
    p.first = {0, best_rounds * per_round, first_cols};
    p.first_tasks = best_rounds * kSweepGroups;
    p.rest = {p.first.rows, rows - p.first.rows, best_cols};
    p.rest_base = 0;
    p.rest_tasks = p.rest.rows * best_cols;
    p.k_chunks = 1;
    p.n_tasks = p.first_tasks + p.rest_tasks;
    return best;
}

// The same sweep in 128 x 64 tiles, one workgroup per task, if that costs less than `large_cost`; true if so (in bf16 plan_narrow
// looks at it again, whichever it is, where K is 320 or more).  A small tile is an eighth of a large one's work and takes n / 8
// of its time where n share a CU.  For bf16 the traffic from L2 makes it up to 2.5 times slower per flop, so there it only
// serves what would leave most of the chip idle.
// Measured, large -> small (us):
//   146 tokens x V 1000, H 64: 14.8 -> 10.4;  x V 5000, H 1024: 35.6 -> 18.5;  x V 32000, H 512: 30.0 -> 26.1 (narrow now);
//   20 x V 152064, H 5120: 478 -> 403 (narrow now).  Where the rule says large: 2500 x V 5000, H 1024: 39.3 (47.4),
//   1000 x V 152064, H 5120: 1297 (2950), and of those that are narrow now 300 x V 32000, H 512: 29.7 (34.2),
//   146 x V 50021, H 1024: 42.2 (57.9)
// fp32, which the matrix cores bound, loses 6 % per flop and wins that back by filling the chip, and always goes this
// way (plan_logprobs): 146 x V 1000, H 64: 28.6 -> 11.0;  500 x V 5000, H 1024: 262 -> 78;  2064 x V 32000, H 1024: 1281 ->
// 1114;  the worst seen, 1000 x V 32000, H 1024: 508 -> 561.
typedef HeadCfg<uint16_t, false, true> SmallShape;
constexpr int kSmallPerCu = SmallShape::kGroupsPerCu;
constexpr double kSmallPart = (double)SmallShape::kTileV * SmallShape::kTileT / ((double)kTile * kTile);
constexpr double kSmallSlower = 2.5;
// What n workgroups that share a CU take for a tile each, in units of a workgroup among three: a CU's only one waits out latencies.  fp32,
// us: 1600 tokens x V 32000, H 1024, 250 tasks of 25 tiles: 955;  1250 of 5: 840;  203 x 15261, H 2240, 240 of 2: 189;  480 of 1: 162.
// (bf16's factor above holds whatever n.)
constexpr double kShareF32[kSmallPerCu + 1] = {0, 1.16, 2.04, 3};
static bool plan_small(HeadParams& p, int64_t M, int64_t V, double large_cost, bool f32 = false) {
    const int64_t rows = (M + SmallShape::kTileT - 1) / SmallShape::kTileT, vts = (V + SmallShape::kTileV - 1) / SmallShape::kTileV;
    double best = large_cost;
    int64_t best_cols = 0;
    for (int64_t s = 1; s <= vts && s <= kMaxSplits; ++s) {
        // (no more partial results than most_triples() has room for)
        if (s > 4 && rows * s * SmallShape::kTileT > kRestTasks * kTile) break;
        const int64_t tasks = rows * s, full = tasks / (kSweepGroups * kSmallPerCu), rest = tasks % (kSweepGroups * kSmallPerCu);
        const double last = rounds_of(rest);
        const double shares = (double)(full * kSmallPerCu) + (f32 ? kShareF32[(int)last] : last);      // tasks in turn on the busiest CU
        const double cost = shares * kSmallPart * ((double)((vts + s - 1) / s) + kTaskCost) * kSmallSlower;
        if (cost < best - 1e-9) { best = cost; best_cols = s; }
    }
    if (best_cols == 0) return false;
    p.M = M;
    p.V = (int)V;
    p.row_tiles = (int)rows;
    p.vocab_tiles = (int)vts;
    p.v_unit = SmallShape::kTileV;
    p.first = {0, 0, 1};
    p.first_tasks = 0;
    p.rest = {0, (int)rows, (int)best_cols};
    p.rest_base = 0;
    p.rest_tasks = (int)(rows * best_cols);
    p.k_chunks = 1;
    p.n_tasks = p.rest_tasks;
    return true;
}

// fp32, and the bf16 rows that the one-token kernel can serve (off a stage or off 16 bytes) with a long H, take the small
// tiles whatever the size (bf16: or narrow ones of up to 128 tokens, plan_narrow, which sum as they do), for the accuracy of
// their sums: the large ones add up all of H one step after the other, which whole-stage bf16 always did.  Error of the
// log-probs against 64 bits, weights of 0.02, rms: H = 5112, 300 tokens, fp32 1.8e-6 in large tiles, 5.0e-7 in small ones (6.1e-7 by
// the one-token kernel); bf16, 1500 tokens, V = 8000, H = 5120 misaligned 7.9e-7, 4.8e-7 (6.1e-7).  At H = 2040 bf16 gives 5.6e-7 in
// large tiles, 6.8e-7 by the one-token kernel.  What that costs, large -> small: 2500 tokens, V = 50000, H = 2104: 0.50 -> 1.09 ms;
// H = 5112: 1.29 -> 2.83 ms; large -> narrow: 16000 tokens, V = 152064, H = 5112: 22.4 -> 38.9 ms (small 108; H = 5120: 17.8 ms).
constexpr int kLongSumH = 2048;
// The forward sweep's schedule; true: in small tiles.  matrix_only: bf16 rows of whole stages at aligned addresses.
static bool plan_logprobs(HeadParams& p, int64_t M, int64_t V, bool bf16, bool matrix_only) {
    const bool only_small = !bf16 || (!matrix_only && p.H > kLongSumH);
    return plan_small(p, M, V, only_small ? 1e300 : plan_sweep(p, M, V), !bf16);
}

// The same sweep in narrow tiles, 256 W rows x 64 n tokens, n = 1 .. 3, where that ends sooner than the division that
// plan_logprobs made in `p`: a few hundred tokens are most of one large tile or several, rounded up, and in small tiles a
// workgroup waits out the latency of every stage.  Columns are ranges of W rows in units of 64 here, so that a call with
// fewer tiles than CUs still spreads W evenly.  Returns n, with `p` set, or 0.
// The times of a stage, a tile and a task on a CU (us; two columns: a W that the caches hold, and one that comes from HBM) are
// fits to 364 sizes (20 .. 1300 tokens, V 1500 .. 152064, H 128 .. 5120; 17 % rms), and the narrow division has to be 5 % better
// by them.  Over 300 of those sizes (H from 320), W in HBM: taken by 132, 1.42 times as fast in the geometric mean, 3 % slower at
// the worst (1300 x V 32000, H 2048: 160 -> 165), and the choice costs 1.1 % more than the best division of each.
// Old division -> narrow, us a call:  100 tokens x V 152064, H 5120: 792 -> 387;  300: 666 -> 573;  20: 423 -> 343;
//   190 x V 32000, H 1024: 57.7 -> 31.1;  500 x V 12000, H 1024: 54.5 -> 27.6;  900 x V 5000, H 2048: 95.1 -> 45.5;
//   1300 x V 12000, H 5120: 246 -> 176.  Where it leaves the old one: 900 x V 152064, H 5120: 1266 (n = 3: 1277);
//   60 x V 32000, H 5120: 97.9 (n = 1: 113).  Below 320 of K it gains nothing.
// fp32 keeps the small tiles (its matrix rate bounds it), and what small tiles served is not given to n = 3, whose sums run over
// all of K: no sum gets longer.  Looked up on every call, on the host: 0.1 us (every number of ranges tried: up to 8).
// Against large tiles the fit holds up to some thousands of tokens (60 sizes of 1300 .. 10000, V from 1000 on: 1.28 times as fast in
// the geometric mean, 1 % slower at the worst); beyond, the division has to be 13 % better by it, and the token rows that
// 256 workgroups sweep at once have to stay in the cache, where every W tile reads them again.  Both sides, us, large -> narrow:
// 16080 x V 1301, H 448: 34.1 -> 32.4;  83412 x 1459, H 320: 146 -> 110;  89178 x 2279, H 1920: 787 -> 739.  By the gain alone refused:
// 9617 x 13530, H 4416: 902 (976);  181148 x 5306, H 1272: 2509 (2745);  98233 x 2697, H 888: 522 (526);  by the rows (409 and 378 MB):
// 45819 x 2169, H 4672: 938 (1099);  81560 x 1053, H 4032: 871 (962).  Small tiles, which long rows at misaligned addresses take
// whatever the size, lose to narrow ones at any (plan_logprobs).
constexpr int64_t kFittedTokens = 8192, kCachedTokens = 192 << 20;
constexpr double kFarGain = 0.87;
constexpr int kNarrowStages = 5;
constexpr double kNarrowGain = 0.95;
constexpr int64_t kCachedW = 128 << 20;            // bytes of W that a pass can expect to find in the 256 MB cache
struct ShapeTime {
    double stage[2], tile, task;
};
constexpr ShapeTime kShapeTime[5] = {              // [n]; 0: small tiles, 4: large ones
    {{0.65, 1.0}, 1.2, 4.0}, {{0.75, 1.45}, 3.0, 5.0}, {{0.95, 1.62}, 3.0, 6.0}, {{1.0, 1.5}, 3.5, 7.0}, {{1.3, 1.65}, 4.5, 8.0}};
static int plan_narrow(HeadParams& p, int64_t M, int64_t V, bool small) {
    if (p.k_tiles < kNarrowStages) return 0;
    const bool from_hbm = V * p.H * 2 > kCachedW;
    auto time_of = [&](int n, double rounds, double tiles) {
        const ShapeTime& t = kShapeTime[n];
        return rounds * (t.task + tiles * (p.k_tiles * t.stage[from_hbm] + t.tile));
    };
    auto in_parts = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
    double best;
    if (small) {
        best = time_of(0, (double)in_parts(p.rest_tasks, kSweepGroups * kSmallPerCu), (double)in_parts(p.vocab_tiles, p.rest.cols));
    } else {
        best = time_of(4, rounds_of(p.rest_tasks), (double)in_parts(p.vocab_tiles, p.rest.cols));
        best += time_of(4, rounds_of(p.first_tasks), (double)in_parts(p.vocab_tiles, p.first.cols));
    }
    best *= small || M <= kFittedTokens ? kNarrowGain : kFarGain;
    constexpr int kUnit = 64;
    const int64_t units = in_parts(V, kUnit);
    int best_n = 0;
    int64_t best_cols = 0;
    for (int n = 1; n <= (small ? 2 : 3); ++n) {
        // Of the divisions that take r rounds of workgroups the finest ends soonest, and the coarsest of those with its
        // tiles per range ends with it.
        const int64_t rows = in_parts(M, 64 * n), most = std::min({units, kRestTasks / rows, kRestTasks * kTile / (rows * 64 * n)});
        for (int64_t r = 1; r <= (int64_t)rounds_of(rows * most); ++r) {
            const int64_t finest = std::min(most, r * kSweepGroups / rows);
            if (finest == 0) continue;
            const int64_t tiles = in_parts(in_parts(units, finest) * kUnit, kTile), s = in_parts(units, tiles * (kTile / kUnit));
            const double t = time_of(n, rounds_of(rows * s), (double)tiles);
            if (t < best - 1e-9) { best = t; best_n = n; best_cols = s; }
        }
    }
    if (best_n == 0) return 0;
    const int64_t rows_at_once = std::min(in_parts(M, 64 * best_n), std::max(kSweepGroups / best_cols, (int64_t)1));
    if (!small && rows_at_once * 64 * best_n * p.H * 2 > kCachedTokens) return 0;
    p.row_tiles = (int)in_parts(M, 64 * best_n);
    p.vocab_tiles = (int)units;
    p.v_unit = kUnit;
    p.first = {0, 0, 1};
    p.first_tasks = 0;
    p.rest = {0, p.row_tiles, (int)best_cols};
    p.rest_tasks = p.n_tasks = p.row_tiles * (int)best_cols;
    return best_n;
}

// The derivative's sweep in large tiles brings W's lines into L2 ahead (head_mfma_kernel) up to this H: between two tiles
// each workgroup stores 128 KB of dz, on an XCD as much as its L2 holds, and the next tile's W is gone from there; with a
// longer H the stores are rarer, and the requests cost more than they give.  The whole backward call, us:
// H 512, 32768 tokens x V 12000: 1284 -> 1246;  H 576, 4096 x 32000: 574 -> 561;  H 1024, 16414 x 32000: 2816 -> 2758;
// H 1536: 4198 -> 4133;  H 2048, 8206 x 32000: 2697 -> 2724, 1300 x 152064: 2609 -> 2581;  H 3584, 8206 x 32000: 4680 -> 4731.
constexpr int kPrefetchH = 1536;

// Plain product of M token-role rows and N W-role rows over K = 64 * k_tiles, columns = W-role tiles.  Whole rounds
// of 256 output tiles first; of the tiles that remain, fewer than a round, each is cut into k_chunks of the
// contraction if that ends sooner.  part_bytes: room for the partial tiles.  In stages: a round of tasks costs kTaskStages besides
// its stages (fill, store, drain), the kernel that adds up the chunks kAddStages, a partial tile kPartStages (written and read
// again, for the most part in the caches).  Kernel times of a call with one output, us, uncut -> as the rule has it (chunks),
// out of the caches:
//   V 5000 x H 128, 900 tokens: d/dh 112 -> 38 (27);  20000 x 512, 400: 380 -> 56 (53);  8000 x 256, 2000: 174 -> 54 (25), d/dW
//   81 -> 62 (8);  35637 x 832, 699: 690 -> 126 (21);  3681 x 3520, 1406: 178 -> 138 (3);  21481 x 64, 3631: 419 -> 85 (17),
//   127 -> 89 (3);  12000 x 2048, 3000: 419 -> 295 (5), 303 -> 285 (2);  32000 x 1024, 16414: 2322 -> 1793 (63).
// Whole by the rule, and for comparison in 2: two rounds instead of one, 9050 x 1088, 1732: d/dW 102 (128);  2439 x 4224, 471:
// 98 (126);  under kLeastCut, 5000 x 128, 900: 46.4 (45.8).
// Contractions of fewer than kLeastCut stages stay whole: their results do not depend on the room (one tile over 17 stages, all
// there is to gain: 35 -> 26).
constexpr double kTaskStages = 6, kAddStages = 6.5, kPartStages = 0.03;
constexpr int kLeastCut = 24;
static void plan_product(HeadParams& p, int64_t M, int64_t N, void* part, size_t part_bytes) {
    const int k_tiles = p.k_tiles;
    p.M = M;
    p.V = (int)N;
    p.row_tiles = (int)((M + kTile - 1) / kTile);
    p.vocab_tiles = (int)((N + kTile - 1) / kTile);
    p.v_unit = kTile;
    p.first = p.rest = {0, p.row_tiles, p.vocab_tiles};
    const int64_t tiles = (int64_t)p.row_tiles * p.vocab_tiles;
    p.first_tasks = (int)(tiles / kSweepGroups * kSweepGroups);
    p.rest_base = p.first_tasks;
    p.rest_tasks = (int)(tiles - p.first_tasks);
    p.k_chunks = 1;
    if (p.rest_tasks > 0 && k_tiles >= kLeastCut) {
        double best = (double)k_tiles + kTaskStages;
        for (int c = 2; c <= kMaxSplits && c <= k_tiles; ++c) {
            const int64_t tasks = (int64_t)c * p.rest_tasks;
            if ((size_t)tasks * kTile * kTile * sizeof(float) > part_bytes) break;
            const double cost = rounds_of(tasks) * ((double)((k_tiles + c - 1) / c) + kTaskStages) + kAddStages + kPartStages * (double)tasks;
            if (cost < best) { best = cost; p.k_chunks = c; }
        }
    }
    p.part_rest = static_cast<float*>(part);
    p.n_tasks = p.first_tasks + p.rest_tasks * p.k_chunks;
}

// Room for them, a multiple of 256.  (It grew with M, and a workspace for many tokens has to serve fewer.)
static size_t arrivals_bytes(int64_t M) { return round_up((size_t)(M / kTile + 64) * 16, 256); }
static_assert(64 * 16 >= kSweepGroups * sizeof(int32_t), "a word for every workgroup");

// A kernel that wants more than 64 KiB of LDS has to be told so once per device.
static bool allow_lds(const void* fn, int lds_bytes) {
    constexpr int kMaxDevices = 64, kMaxKernels = 16;
    static std::atomic<const void*> done[kMaxDevices][kMaxKernels];
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) return false;
    std::atomic<const void*>* row = dev < kMaxDevices ? done[dev] : nullptr;
    int free_slot = -1;
    if (row) {
        for (int i = 0; i < kMaxKernels; ++i) {
            const void* seen = row[i].load(std::memory_order_acquire);
            if (seen == fn) return true;
            if (!seen && free_slot < 0) free_slot = i;
        }
    }
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes) != hipSuccess) return false;
    if (row && free_slot >= 0) row[free_slot].store(fn, std::memory_order_release);   // (a lost race only repeats the call)
    return true;
}

// Launch one sweep: large tiles one workgroup per CU, which re-align if there is more than one round; small and narrow tiles one
// workgroup per task, as many for every XCD, which takes consecutive tasks (small tiles dealt out one by one, us: fp32, 2064
// tokens x V 32000, H 1024: 1214, so: 1147; bf16, 1500 x 8000, H 5112: 322, 306).  Only the derivative's small tiles of several
// token tiles are dealt out, whose stores go slower where every XCD has a range of V of its own, us: 358 tokens x V 11732,
// H 192: 21.0, so: 17.2;  400 x 10000, H 192: 19.9, 16.8;  700 x 6000, H 256: 21.8, 19.3;  120 x 13687, H 384: 14.5, 13.7;  436 x 987,
// H 64: 7.6, 7.8; of one token tile, 34 x 24566, H 128: 9.6, 9.9.  A device that does not report 256 compute
// units (a partition of the chip, another chip) is refused: the sweep would still be correct there, but its workgroups would
// take turns instead of running side by side.
template <class C, template <class> class Epi>
static int launch_sweep(HeadParams& p, void* arrivals, hipStream_t s) {
    if (device_compute_units() != kSweepGroups) return TPPO_ERR_LAUNCH;
    if (C::kLdsBytes > 64 * 1024 && !allow_lds(reinterpret_cast<const void*>(head_mfma_kernel<C, Epi>), C::kLdsBytes))
        return TPPO_ERR_LAUNCH;
    static_assert(C::kSmall || C::kNarrow || (kTile == C::kTileV && kTile == C::kTileT), "the schedule counts in these tiles");
    p.arrivals = !C::kSmall && !C::kNarrow && p.n_tasks > kSweepGroups ? static_cast<int32_t*>(arrivals) : nullptr;
    constexpr int kMostGroups = 1 << 20;                            // (beyond that, several tasks per workgroup)
    const int tasks = (p.n_tasks + 7) / 8 * 8;
    const int groups = !C::kSmall && !C::kNarrow ? kSweepGroups : tasks < kMostGroups ? tasks : kMostGroups;
    hipLaunchKernelGGL((head_mfma_kernel<C, Epi>), dim3(groups), dim3(C::kThreads),
                       C::kLdsBytes, s, p);
    return launch_result();
}

template <bool RAGGED, template <class> class Epi>
static int launch_narrow(int n, HeadParams& p, hipStream_t s) {
    return n == 1   ? launch_sweep<HeadCfg<uint16_t, RAGGED, false, 0, 1>, Epi>(p, nullptr, s)
           : n == 2 ? launch_sweep<HeadCfg<uint16_t, RAGGED, false, 0, 2>, Epi>(p, nullptr, s)
                    : launch_sweep<HeadCfg<uint16_t, RAGGED, false, 0, 3>, Epi>(p, nullptr, s);
}

}  // namespace tppo
