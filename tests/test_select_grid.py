"""The token filter's one launch (csrc/select.hip, host side): all of its workgroups have a place on the chip at once."""
import os
import subprocess

from test_head_routes import HIPCC, ROOT

PROGRAM = r"""
#include <cstdio>
#include "select.hip"
namespace tppo { int device_compute_units() { return 256; } }
int main() {
    for (int plan = 0; plan < 2; ++plan)
        for (int64_t B : {1, 128, 129, 1024})
            for (int64_t most : {0, 1, 300, 511, 512, 10000}) {
                const int parts = tppo::list_parts(plan, B), workers = tppo::one_launch_workers(most, parts);
                printf("%ld %d %d\n", (long)most, parts, workers);
            }
}
"""


def test_no_workgroup_without_a_place(tmp_path):
    (tmp_path / "grid.hip").write_text(PROGRAM)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2506_15050_amd", "csrc"), str(tmp_path / "grid.hip"), "-o", str(tmp_path / "grid")],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    out = subprocess.run([str(tmp_path / "grid")], check=True, stdout=subprocess.PIPE, text=True).stdout
    rows = [tuple(map(int, line.split())) for line in out.splitlines()]
    assert len(rows) == 48
    for most, parts, workers in rows:
        # 1024 threads each: two on each of 256 CUs
        assert parts + workers <= 512 and workers == min(most, 512 - parts)
