"""Log-prob sweeps in narrow tiles (256 W rows x 64, 128 or 192 tokens): which calls take them (the rule itself,
csrc/head_tile.h, run on the host) and their results at the edges of tiles, of W ranges and of the last K stage."""
import os
import subprocess

import numpy as np
import pytest

from test_gpu_parity import _bf16_case, check_logprob_grads, dev, host, ofast, tp  # noqa: F401
from test_head_routes import HIPCC, ROOT
from paper_2506_15050_amd import synth

# (tokens, vocabulary, hidden size): (64-token blocks of a tile, W ranges)
NARROW = {
    (65, 30011, 1024): (1, 118),                   # one token beyond a tile, W ranges of three and of four units
    (385, 5000, 832): (1, 20),
    (700, 5000, 1024): (1, 20),
    (2500, 1011, 640): (1, 4),                     # 40 token tiles
    (257, 20033, 1024): (2, 79),
    (500, 12000, 320): (2, 47),                    # the shortest K
    (1025, 7001, 704): (2, 28),
    (900, 20001, 576): (3, 40),
    (16080, 1301, 448): (3, 3),                    # many tokens
    (1300, 12007, 576): (3, 24),                   # ranges of two tiles, the second short
}
NARROW_RAGGED = {
    (385, 5000, 840): (1, 20),
    (1300, 4003, 2120): (2, 16),                   # too long for one sum over K
    (450, 9000, 329): (2, 36),                     # rows copied to 336
    (300, 20000, 333): (2, 79),
    (1300, 12007, 584): (3, 24),
    (2500, 9000, 1000): (3, 18),
}
NARROW_TOO = {(16000, 152064, 5112): (2, 2), (20, 152064, 5120): (1, 198)}      # (too large for a test's oracle)
# the derivative's large tiles, where they bring W's lines ahead: one, two, three and more token tiles beside each other, one and
# several stages, a short last tile of W
LARGE_AHEAD = [(250, 60001, 64), (512, 33000, 64), (700, 33000, 64), (1100, 9001, 192), (8100, 2047, 1536)]
NOT = [(500, 12000, 256), (942, 152064, 5120), (60, 32000, 5120), (400, 32000, 1024), (15000, 32000, 1024),
       (9617, 13530, 4416), (181148, 5306, 1272),      # many tokens: too little gained by the model
       (45819, 2169, 4672), (81560, 1053, 4032)]       # ... or more token rows at once than the cache holds

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "head_tile.h"
namespace tppo { int device_compute_units() { return 256; } }
int main(int argc, char** argv) {
    for (int i = 1; i + 2 < argc; i += 3) {
        tppo::HeadParams p = {};
        p.H = (atoi(argv[i + 2]) + 7) / 8 * 8;
        p.k_tiles = (p.H + 63) / 64;
        const long M = atol(argv[i]), V = atol(argv[i + 1]);
        const bool small = tppo::plan_logprobs(p, M, V, true, p.H % 64 == 0);
        const int n = tppo::plan_narrow(p, M, V, small);
        const bool ahead = !small && n == 0 && p.H <= tppo::kPrefetchH;
        printf("%d %d %d %d %d\n", n, p.rest.cols, n == 0 || p.rest.rows == (M + 64 * n - 1) / (64 * n), p.n_tasks, ahead);
    }
}
"""


# the rule's model with every number of ranges tried, over random calls; prints how many are divided otherwise and the time both take
SEARCH = r"""
#include <chrono>
#include <cmath>
#include <cstdio>
#include <random>
#include "head_tile.h"
namespace tppo {
int device_compute_units() { return 256; }
static int search(const HeadParams& p, int64_t M, int64_t V, bool small, int64_t& cols) {
    cols = 0;
    if (p.k_tiles < kNarrowStages) return 0;
    auto parts = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
    auto time_of = [&](int n, double rounds, double tiles) {
        const ShapeTime& t = kShapeTime[n];
        return rounds * (t.task + tiles * (p.k_tiles * t.stage[V * p.H * 2 > kCachedW] + t.tile));
    };
    double best;
    if (small) {
        best = time_of(0, (double)parts(p.rest_tasks, kSweepGroups * kSmallPerCu), (double)parts(p.vocab_tiles, p.rest.cols));
    } else {
        best = time_of(4, rounds_of(p.rest_tasks), (double)parts(p.vocab_tiles, p.rest.cols)) +
               time_of(4, rounds_of(p.first_tasks), (double)parts(p.vocab_tiles, p.first.cols));
    }
    best *= small || M <= kFittedTokens ? kNarrowGain : kFarGain;
    int found = 0;
    for (int n = 1; n <= (small ? 2 : 3); ++n) {
        const int64_t rows = parts(M, 64 * n), units = parts(V, 64);
        for (int64_t s = 1; s <= units && rows * s <= kRestTasks && rows * s * 64 * n <= kRestTasks * kTile; ++s) {
            const double t = time_of(n, rounds_of(rows * s), (double)parts(parts(units, s) * 64, kTile));
            if (t < best - 1e-9) { best = t; found = n; cols = s; }
        }
    }
    if (found == 0 || small) return found;
    const int64_t at_once = std::min(parts(M, 64 * found), std::max(kSweepGroups / cols, (int64_t)1)) * 64 * found;
    return at_once * p.H * 2 > kCachedTokens ? 0 : found;
}
}
int main() {
    using namespace tppo;
    using std::chrono::steady_clock;
    std::mt19937_64 bits(7);
    auto between = [&](double a, double b) { return std::lround(a * std::pow(b / a, (bits() >> 11) * 0x1p-53)); };
    int otherwise = 0, taken = 0;
    double times[2] = {0, 0};
    for (int i = 0; i < 20000; ++i) {
        const long M = between(1, 200000), V = between(1, 152064), H = between(8, 5200);
        HeadParams p = {};
        p.H = (int)(H + 7) / 8 * 8;
        p.k_tiles = (p.H + 63) / 64;
        const bool small = plan_logprobs(p, M, V, true, p.H % 64 == 0);
        int64_t cols;
        const auto t0 = steady_clock::now();
        const int want = search(p, M, V, small, cols);
        const auto t1 = steady_clock::now();
        const int n = plan_narrow(p, M, V, small);
        const auto t2 = steady_clock::now();
        times[0] += std::chrono::duration<double>(t1 - t0).count();
        times[1] += std::chrono::duration<double>(t2 - t1).count();
        otherwise += n != want || (n && p.rest.cols != cols);
        taken += n != 0;
    }
    printf("%d %d %g %g\n", otherwise, taken, times[0], times[1]);
}
"""


def compiled(at, program):
    at.with_suffix(".hip").write_text(program)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2506_15050_amd", "csrc"), str(at.with_suffix(".hip")), "-o", str(at)],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    return str(at)


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    program = compiled(tmp_path_factory.mktemp("narrow") / "narrow", PROGRAM)

    def run(shapes):
        out = subprocess.run([program, *(str(x) for s in shapes for x in s)], check=True, stdout=subprocess.PIPE,
                             text=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return run


def test_which_calls(rule):
    for table in (NARROW, NARROW_RAGGED, NARROW_TOO):
        got = dict(zip(table, rule(table)))
        assert {s: g[:2] for s, g in got.items()} == table
        # every token has a tile, and the partial results stay within what a workspace holds
        assert all(g[2] and g[3] <= 1024 and g[3] * 64 * g[0] <= 1024 * 256 for g in got.values())
    assert [g[0] for g in rule(NOT)] == [0] * len(NOT)
    assert all(g[4] for g in rule(LARGE_AHEAD))


def test_the_rule_looks_at_few_divisions(tmp_path):
    """It finds what trying every number of ranges finds, in a fraction of the time (each call pays for it on the host)."""
    out = subprocess.run([compiled(tmp_path / "search", SEARCH)], check=True, stdout=subprocess.PIPE, text=True).stdout.split()
    otherwise, taken, every, rule_itself = int(out[0]), int(out[1]), float(out[2]), float(out[3])
    assert otherwise == 0 and taken > 500 and rule_itself < every / 2


@pytest.mark.gpu
@pytest.mark.parametrize("M,V,H", [*NARROW, *NARROW_RAGGED])
def test_logprobs(tp, M, V, H):
    rng = np.random.default_rng(M + V + H)
    hidden = synth.f32_to_bf16_bits(rng.normal(size=(301, H)).astype(np.float32))
    w = synth.f32_to_bf16_bits((rng.normal(size=(V, H)) / np.sqrt(H)).astype(np.float32))
    rows, targets = rng.integers(0, 301, size=M), (np.arange(M) * 7 + V - 1) % V
    firsts = np.arange(64, V, 64)[: M // 2]                # sampled tokens on both sides of where a range of W may begin
    targets[: len(firsts)], targets[M - len(firsts):] = firsts, firsts - 1
    out = dev(rng.permutation(M + 5)[:M].astype(np.int32))
    args = (dev(hidden), dev(w), dev(rows.astype(np.int32)), dev(targets.astype(np.int32)))
    ref, ref_lse = ofast.token_logprobs(hidden, w, rows, targets)
    at = host(out)
    for n in (M, M - M // 3 - 1):                          # the device's own count: token tiles cut short and left out
        st = tp.new_status("cuda")
        logp, lse = tp.tppo_token_logprobs(*args, m_actual=dev(np.array([n], np.int64)), out_index=out, out_size=M + 5, status=st)
        assert int(host(st)[0]) == 0
        # exact products summed in fp32 over H and V, logits of size about 5: a few times 2^-24 * 8
        assert np.abs(host(logp)[at][:n] - ref[:n]).max() <= 1e-5 and np.abs(host(lse)[at][:n] - ref_lse[:n]).max() <= 1e-5


@pytest.mark.gpu
@pytest.mark.parametrize("M,V,H", [(385, 5000, 832), (500, 12000, 320), (1300, 12007, 576)])
def test_grads(tp, M, V, H):
    check_logprob_grads(tp, *_bf16_case(M, V, H, seed=M + V))


@pytest.mark.gpu
@pytest.mark.parametrize("M,V,H", LARGE_AHEAD)
def test_grads_large_tiles_prefetch(tp, M, V, H):
    """The lines brought in ahead end with W, and with the task."""
    check_logprob_grads(tp, *_bf16_case(M, V, H, seed=M + V))
