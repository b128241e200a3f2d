"""How the backward pass's products divide their output tiles (csrc/head_tile.h, plan_product, run on the host): every K
step of every tile belongs to exactly one task, the partial tiles fit their room, and room beyond the recommended
workspace's changes nothing."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "head_tile.h"
namespace tppo { int device_compute_units() { return 256; } }
using namespace tppo;
static int check(long M, long N, int k_tiles, size_t room) {
    HeadParams p = {};
    p.k_tiles = k_tiles;
    plan_product(p, M, N, nullptr, room);
    const long tiles = (M + 255) / 256 * ((N + 255) / 256);
    bool good = p.first_tasks % 256 == 0 && p.first_tasks + p.rest_tasks == tiles && p.rest_tasks < 256 &&
                p.n_tasks == p.first_tasks + p.rest_tasks * p.k_chunks && p.k_chunks >= 1 && p.k_chunks <= k_tiles;
    if (p.k_chunks > 1) good = good && k_tiles >= 24 && (size_t)p.rest_tasks * p.k_chunks * 256 * 256 * 4 <= room;
    // the kernels' own tasks: a tile's steps follow each other, in chunk order and without a gap, and a partial tile lies where
    // the adding kernel looks for it, under the output tile that it is of
    std::vector<int> at(tiles, 0);
    for (int t = 0; good && t < p.n_tasks; ++t) {
        const Task x = task_at<true>(p, t, k_tiles);
        const long rows = (M + 255) / 256, tile = x.col * rows + x.row;
        good = x.row >= 0 && x.row < rows && tile >= 0 && tile < tiles && x.k_begin == at[tile] && x.k_tiles > 0 &&
               x.v_begin == x.col * 256 && x.v_end == std::min(N, x.v_begin + 256l);
        if (!good) break;
        at[tile] = x.k_begin + x.k_tiles;
        if (x.rest) {
            const int id = x.part % p.rest_tasks;
            const Task sum = task_at<true>(p, p.first_tasks + id, 1);
            good = good && x.part == t - p.first_tasks && x.part < p.rest_tasks * p.k_chunks && sum.row == x.row && sum.col == x.col;
        }
    }
    for (long i = 0; i < tiles; ++i) good = good && at[i] == k_tiles;
    if (!good) printf("M %ld N %ld k %d room %zu: first %d rest %d chunks %d\n", M, N, k_tiles, room,
                                         p.first_tasks, p.rest_tasks, p.k_chunks);
    return p.k_chunks > 1;
}
int main() {
    const long sizes[] = {1, 63, 256, 257, 700, 2049, 9000, 33000, 152064};
    const int depths[] = {1, 2, 23, 24, 25, 64, 257, 500, 2376};
    int cut = 0;
    for (long M : sizes) for (long N : {64l, 320l, 1024l, 5120l, 5184l}) for (int k : depths)
        for (size_t room : {(size_t)0, (size_t)1 << 18, (size_t)5 << 18, (size_t)1 << 27}) cut += check(M, N, k, room);
    printf("cut %d\n", cut > 50);
}
"""


ROOM = r"""
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include "head_bwd.hip"
namespace tppo { int device_compute_units() { return 256; } }
using namespace tppo;
int main() {
    srand48(7);
    int cut = 0;
    for (int i = 0; i < 10000; ++i) {
        const int64_t M = 1 + (int64_t)exp(drand48() * log(i % 10 ? 2e4 : 3e5)), V = 1 + (int64_t)exp(drand48() * log(1.6e5));
        const int64_t H = 64 * (1 + lrand48() % 80);
        const size_t asked = tppo_token_logprobs_backward_workspace_bytes(M, H, V, TPPO_BF16);
        const BwdLayout L = bwd_layout(H, V, std::min((M + 255) / 256 * 256, kBwdChunkDefault));
        const size_t room = std::min(kPartBytes, asked - L.off_part);
        bool good = asked >= L.total;
        for (int64_t m0 = 0; m0 < M; m0 += L.chunk)
            for (int product = 0; product < 2; ++product) {
                HeadParams p = {}, q = {};
                plan_bwd_product(p, product, std::min(M - m0, L.chunk), H, V, nullptr, room);
                plan_bwd_product(q, product, std::min(M - m0, L.chunk), H, V, nullptr, kPartBytes);
                good = good && p.k_chunks == q.k_chunks;
                cut += p.k_chunks > 1;
            }
        if (!good) printf("M %ld V %ld H %ld\n", (long)M, (long)V, (long)H);
    }
    printf("cut %d\n", cut > 1000);
}
"""


def check(tmp_path, program):
    (tmp_path / "plan.hip").write_text(program)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2506_15050_amd", "csrc"), str(tmp_path / "plan.hip"), "-o", str(tmp_path / "plan")],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    assert subprocess.run([str(tmp_path / "plan")], check=True, stdout=subprocess.PIPE, text=True).stdout.split("\n") == ["cut 1", ""]


def test_every_step_in_one_task(tmp_path):
    check(tmp_path, PROGRAM)


def test_more_room_divides_no_other_way(tmp_path):
    check(tmp_path, ROOM)
