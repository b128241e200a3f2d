"""Which sets a token of the loss passes belongs to (csrc/losses.hip, token_sets, run on the host): every thread of every
workgroup against the definition, and no thread reads the sequences' words in a frame that the workgroup has not fetched
them for, batches that end in empty windows among them.  Of batches that one fetch holds, also with all sequences fetched from the
first one on, as by grids of few workgroups."""
import os
import subprocess

from test_head_routes import HIPCC, ROOT

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <sys/mman.h>
#include <vector>
#include "plan_build.h"
#include "losses.hip"
namespace tppo {
uint32_t next_call_tag() { return 1; }
int launch_plan_build(const int32_t*, const int32_t*, const int32_t*, int64_t, int64_t, int64_t, void*, int32_t*, hipStream_t) { return 0; }
}
using namespace tppo;
typedef std::vector<int> Ints;
static const MoreSeqs* nobody;                                      // reading it ends the program
static int frames_with_more, frames_of_all;
static void check(const Ints& win, const Ints& keep, const Ints& done) {
    const int B = (int)win.size();
    Ints off(B + 1, 0);
    for (int i = 0; i < B; ++i) off[i + 1] = off[i] + win[i];
    const int n = off[B];
    std::vector<FrameDesc> frames(n / kTileTokens + B + 1);
    Plan pl = {};
    pl.frames = frames.data();
    pl.cap = (int)frames.size();
    for (int i = 0; i < B; ++i) {
        const int tiles = window_tiles(off[i], win[i]);
        for (int l = 0; l < tiles; ++l)
            note_frame(pl, make_tile(i, off[i], win[i], tiles, l), off[i], win[i], true, keep[i], done[i] != 0,
                       next_sequence(i, off[i], off[i + 1], (const int*)off.data(), keep.data(), done.data(), true, B, n));
    }
    Ints pol(n, 0), val(n, 0);
    for (int i = 0; i < B; ++i)
        for (int t = off[i]; t < off[i + 1]; ++t) pol[t] = t - off[i] < keep[i], val[t] = done[i] != 0;
    LossParams p = {};
    p.resp_off = off.data(); p.keep_len = keep.data(); p.done = done.data(); p.B = B; p.n_resp = n;
    MoreSeqs fetched, all;
    for (int item = 0; item * 4 * kLossThreads < n; ++item) {
        const FrameDesc d = frames[item / kLossParts];
        const bool more = has_more(p, d, item);
        frames_with_more += more;
        const bool one_fetch = B <= kLossThreads;                   // (all_ahead)
        frames_of_all += more && one_fetch;
        auto fetch = [&](MoreSeqs& into, int from) {                // (keep_meta)
            for (int w = 0; w < kLossThreads / kWave; ++w) into.in_frame[w] = 0;
            for (int tid = 0; tid < kLossThreads; ++tid) {
                const SeqMeta x = load_meta(p, from + tid);
                into.in_frame[tid / kWave] += from + tid < B && x.lo < (item + 1) * (4 * kLossThreads);
                into.seq[tid] = kept_words(x);
            }
        };
        fetch(fetched, d.seg2 + 1);
        fetch(all, 0);
        for (int tid = 0; tid < kLossThreads; ++tid) {
            for (const TokenSets& ts : {token_sets<true>(p, d, more, more ? fetched : *nobody, item, tid, true, true),
                                        token_sets<true>(p, d, more, more ? fetched : *nobody, item, tid, true, true, d.seg2 + 1),
                                        one_fetch ? token_sets<true>(p, d, more, more ? all : *nobody, item, tid, true, true, 0)
                                                  : token_sets<false>(p, d, false, *nobody, item, tid, true, true),
                                        token_sets<false>(p, d, false, *nobody, item, tid, true, true)}) {
                int want_pol = 0, want_val = 0;
                for (int e = 0; e < ts.n_tok; ++e) want_pol |= pol[ts.first + e] << e, want_val |= val[ts.first + e] << e;
                if (ts.pol != want_pol || ts.val != want_val) {
                    printf("B %d n %d item %d thread %d: %x %x, not %x %x\n", B, n, item, tid, ts.pol, ts.val, want_pol, want_val);
                    exit(1);
                }
            }
        }
    }
}
static Ints repeat(Ints head, int n, int x) {
    head.insert(head.end(), n, x);
    return head;
}
int main() {
    nobody = static_cast<const MoreSeqs*>(mmap(nullptr, 1 << 20, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0));
    std::vector<Ints> layouts = {{700, 0}, {700, 1, 0}, {700, 0, 0}, {1500, 3, 0, 0}, {1024, 5, 0}, {1024, 0}, {4, 0}, {700},
                                 repeat({5, 3}, 300, 0), repeat({700}, 300, 0), repeat({700, 1}, 70, 0), repeat({1, 1}, 600, 2),
                                 repeat({1023, 1}, 300, 1), repeat({}, 1500, 1),
                                 repeat({}, 255, 1), repeat({}, 256, 1), repeat({}, 257, 1), repeat({}, 255, 9), repeat({}, 256, 9),
                                 repeat({3000}, 255, 9), repeat({3000}, 254, 2), repeat({0, 0, 700}, 253, 4), repeat(repeat({}, 200, 0), 56, 9),
                                 repeat(repeat(repeat({}, 100, 0), 90, 3), 66, 0), repeat(repeat(repeat({5}, 200, 0), 54, 7), 1, 0),
                                 repeat(repeat(repeat({}, 250, 0), 5, 400), 1, 1), repeat(repeat({2000}, 127, 0), 128, 5)};
    srand(3);
    for (int k = 0; k < 300; ++k) {                                 // runs of empty, short and long windows, often at the end
        Ints win = {1 + rand() % 900};
        for (int run = rand() % 8; run >= 0; --run) {
            const int most[] = {1, 1, 4, 40, 1500}, m = most[rand() % 5], n = 1 + rand() % (m < 40 ? 300 : 6);
            for (int i = 0; i < n; ++i) win.push_back(rand() % m);
        }
        layouts.push_back(win);
    }
    for (const Ints& win : layouts) {
        Ints keep, done;
        for (int w : win) {
            done.push_back(rand() % 2);
            keep.push_back(done.back() || rand() % 2 ? w : rand() % (w + 1));
        }
        check(win, keep, done);
    }
    printf("%d layouts, frames with more: %d %d\n", (int)layouts.size(), frames_with_more > 100, frames_of_all > 100);
}
"""

# workgroups of the largest and other batches, of the product's grids and (argument: built for tuning) of grids whose size the
# environment gives
GROUPS = r"""
#include "losses.hip"
#include <cstdio>
#include <cstdlib>
namespace tppo {
uint32_t next_call_tag() { return 1; }
int launch_plan_build(const int32_t*, const int32_t*, const int32_t*, int64_t, int64_t, int64_t, void*, int32_t*, hipStream_t) { return 0; }
}
int main() {
    for (const char* groups : {"", "1", "2", "100", "127", "128", "1024", "2048", "2049", "-5"}) {
        setenv("TPPO_LOSS_GROUPS", groups, 1);
        for (int64_t n : {(int64_t)1, (int64_t)1 << 20, ((int64_t)1 << 24) - 1, (int64_t)1 << 24, ((int64_t)1 << 24) + 1, (int64_t)INT32_MAX})
            for (bool grad : {false, true}) printf("%s,%ld,%d\n", groups, (long)n, tppo::loss_groups(n, grad));
    }
}
"""


def compiled(at, program, *flags):
    at.with_suffix(".hip").write_text(program)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", *flags, "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2506_15050_amd", "csrc"), str(at.with_suffix(".hip")), "-o", str(at)],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    return str(at)


def test_a_workgroups_tokens_can_be_counted_in_fp32(tmp_path):
    for flags in ((), ("-DTPPO_TUNING",)):
        out = subprocess.run([compiled(tmp_path / "groups", GROUPS, *flags)], check=True, stdout=subprocess.PIPE, text=True, timeout=60).stdout
        rows = [line.split(",") for line in out.splitlines()]
        assert len(rows) == 120
        for forced, n, groups in ((f, int(n), int(g)) for f, n, g in rows):
            frames = -(-n // 1024)
            assert 1 <= groups <= min(frames, 2048) and -(-frames // groups) * 1024 <= 1 << 24, (forced, n, groups)
            if flags and forced.isdigit() and 128 <= int(forced) <= 2048:
                assert groups == min(frames, int(forced))
            if not flags:
                assert groups == min(frames, 1024)


def test_lookup_reads_what_was_fetched(tmp_path):
    ran = subprocess.run([compiled(tmp_path / "lookup", PROGRAM)], stdout=subprocess.PIPE, text=True, timeout=120)
    assert ran.returncode == 0 and ran.stdout == "327 layouts, frames with more: 1 1\n", (ran.returncode, ran.stdout)
