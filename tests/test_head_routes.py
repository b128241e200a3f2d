"""Which tiles and which division of the work the log-prob sweep takes: the rules
themselves (csrc/head_tile.h, host side) in the order in which a call asks them,
run at the sizes that the GPU tests rely on to reach a path.  A change of a rule
that moves one of them shows here.  (Narrow tiles: test_gpu_head_narrow.py.)"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# (tokens, vocabulary, hidden size): (token tiles, columns) of the whole rounds, of the rest
LARGE_WHOLE = {
    (200, 152064, 64): ((0, 4), (1, 198)),         # one token tile
    (130, 131072, 64): ((0, 4), (1, 256)),         # ... against as many vocabulary ranges as there may be
    (513, 65281, 64): ((0, 4), (3, 256)),          # three tasks per workgroup, a last vocabulary tile of one entry
    (1024, 40961, 64): ((0, 4), (4, 54)),          # whole token tiles only
    (17000, 4000, 64): ((64, 4), (3, 16)),         # a whole round and a finely cut rest
    (33000, 1100, 64): ((64, 4), (65, 3)),         # a whole round and a rest of nearly another, 5 vocabulary tiles
    (1000, 32000, 1024): ((0, 4), (4, 63)),        # K stages enough for narrow tiles, which gain too little here
}
LARGE_WHOLE_ELSEWHERE = {                          # shapes of other tests
    (16500, 600, 64): ((0, 2), (65, 3)),           # no whole round although there could be one
    (33000, 300, 64): ((0, 2), (129, 1)),
    (66000, 200, 64): ((256, 1), (2, 1)),          # one vocabulary tile: a round of 256 token tiles
    (18600, 2048, 64): ((0, 4), (73, 3)),
    (21000, 1100, 128): ((0, 4), (83, 3)),
    (4200, 9000, 64): ((0, 4), (17, 12)),
}
LARGE_RAGGED = {                                   # bf16 rows off a stage of 64
    (300, 20000, 72): ((0, 4), (2, 79)),
    (700, 30000, 8): ((0, 4), (3, 59)),            # a stage that is mostly zeros
    (300, 20000, 203): ((0, 4), (2, 79)),          # rows copied to 208
    (1000, 32000, 1000): ((0, 4), (4, 63)),        # 16 K stages
    (600, 60000, 1013): ((0, 4), (3, 79)),         # ... of rows copied to 1016
    (17000, 4000, 392): ((64, 4), (3, 16)),        # 7 stages, whole rounds and a rest
    (18600, 2048, 200): ((0, 4), (73, 3)),
    (17000, 4000, 136): ((64, 4), (3, 16)),
    (33000, 1100, 72): ((64, 4), (65, 3)),
}
SMALL_WHOLE = {
    (5, 70000, 64): (1, 183),
    (1030, 3000, 64): (17, 12),
    (1, 256, 64): (1, 2), (37, 1000, 128): (1, 8), (300, 1000, 256): (5, 8), (513, 2049, 192): (9, 17),
    (256, 512, 64): (4, 4),
    (64, 32000, 1024): (1, 250), (20, 1500, 320): (1, 12),       # K stages enough for narrow tiles
}
SMALL_RAGGED = {
    (57, 333, 72): (1, 3),
    (1500, 8000, 5120): (24, 21),                  # long rows at misaligned addresses, whatever the size
    (1500, 8000, 2112): (24, 21), (300, 4000, 5112): (5, 32), (300, 4000, 5100): (5, 32),
}
SMALL_FP32 = {(2064, 32000, 1024): (33, 23), (300, 32000, 64): (5, 50)}

# fp32 in small tiles, (token tiles, columns): up to 512 tasks, two workgroups to a CU, and more
FP32_FEW = {(1500, 9000, 72): (24, 18), (2100, 3000, 64): (33, 12), (203, 15261, 64): (4, 120)}
FP32_MANY = {(1400, 4097, 64): (22, 33), (1400, 4097, 72): (22, 33), (520, 8300, 64): (9, 65)}

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "head_tile.h"
namespace tppo { int device_compute_units() { return 256; } }
int main(int argc, char** argv) {
    for (int i = 1; i + 4 < argc; i += 5) {
        tppo::HeadParams p = {};
        p.H = (atoi(argv[i + 2]) + 7) / 8 * 8;
        const long M = atol(argv[i]), V = atol(argv[i + 1]);
        const bool bf16 = atoi(argv[i + 3]), small = tppo::plan_logprobs(p, M, V, bf16, atoi(argv[i + 4]));
        p.k_tiles = (p.H + 63) / 64;
        const int narrow = bf16 ? tppo::plan_narrow(p, M, V, small) : 0;
        printf("%d %d %d %d %d\n", narrow ? 2 : small, p.first_tasks ? p.first.rows : 0, p.first.cols, p.rest.rows, p.rest.cols);
    }
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    at = tmp_path_factory.mktemp("routes")
    (at / "routes.hip").write_text(PROGRAM)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2506_15050_amd", "csrc"), str(at / "routes.hip"), "-o", str(at / "routes")],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)

    def run(shapes, bf16, whole):
        args = [str(x) for s in shapes for x in (*s, int(bf16), int(whole))]
        out = subprocess.run([str(at / "routes"), *args], check=True, stdout=subprocess.PIPE, text=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return run


@pytest.mark.parametrize("table,whole", [(LARGE_WHOLE, True), (LARGE_WHOLE_ELSEWHERE, True), (LARGE_RAGGED, False)])
def test_large_tiles(rule, table, whole):
    got = {s: ((f_rows, f_cols), (r_rows, r_cols)) if tiles == 0 else tiles
           for s, (tiles, f_rows, f_cols, r_rows, r_cols) in zip(table, rule(table, True, whole))}
    assert got == table


@pytest.mark.parametrize("table,bf16,whole", [(SMALL_WHOLE, True, True), (SMALL_RAGGED, True, False), (SMALL_FP32, False, True)])
def test_small_tiles(rule, table, bf16, whole):
    got = {s: (rows, cols) if tiles == 1 else tiles for s, (tiles, _, _, rows, cols) in zip(table, rule(table, bf16, whole))}
    assert got == table


def test_fp32_tasks(rule):
    for table, few in ((FP32_FEW, True), (FP32_MANY, False)):
        for s, (rows, cols) in table.items():
            assert rule([s], False, s[2] % 32 == 0) == [(1, 0, 1, rows, cols)] and (rows * cols <= 512) == few
