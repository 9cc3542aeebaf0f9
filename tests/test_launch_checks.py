"""What the launchers refuse before any device call, in plans that no workspace of a real GPU leads to."""
import os
import subprocess

import pytest

import paper_2402_14118_amd as mm

CSRC = os.path.join(os.path.dirname(mm.__file__), "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include <cstdio>
#include "mmm_internal.h"
int main()
{
    mmm_maps m{};
    m.M = 1LL << 22; m.K = 128; m.N = 1LL << 22; m.bw = 16; m.KBA = 1; m.NG = m.N / 16;
    mmm_plan p{};
    p.split_k = 1; p.chunks_total = p.chunks_per_split = 1; p.panel = 1 << 16;
    p.tiles_m = 1 << 16; p.tiles_n = 1 << 16;                  // 2^32 tiles: none, in 32 bits
    p.workgroups = (int64_t)p.tiles_m * p.tiles_n;
    std::printf("%d\n", (int)(mmm_launch_matmul(&m, p, MMM_F32, nullptr, m.N, 0, nullptr, 0, nullptr) == hipErrorInvalidValue));
    return 0;
}
"""


GROUPS = r"""
#include <cstdio>
#include "mmm_internal.h"
int main()
{
    int bad = 0, waves = 0;
    for (int32_t v = 0; v < mmm_variant_count(); ++v)
        for (int64_t N = 8; N <= 4096; N += 8)
            for (int bw : {8, 32}) {
                if (N % bw != 0) continue;
                const int width = bw == 32 ? 2 : 1, groups = (int)((N + 15) / 16), tile = mmm_variant(v).TN / 16;
                for (int g = 0; g < (groups + tile - 1) / tile * tile; g += width, ++waves) {   // the first group of each wave of the grid
                    const int walked = mmm_walked_group(g, groups, width);
                    bad += walked < 0 || walked + width > groups || (g < groups && walked != g);
                }
            }
    std::printf("%d %d\n", bad, (int)(waves > 0));
    return 0;
}
"""

PLACES = r"""
#include <cstdio>
#include <vector>
#include "mmm_internal.h"
int main()
{
    int bad = 0;
    for (uint32_t units = 1; units <= 300; units += units < 20 ? 1 : 7)
        for (uint32_t blocks = 1; blocks <= 33; ++blocks)           // below each other
            for (uint32_t per : {1u, 2u, 6u, 8u}) {                // for each workgroup, the last row of them less
                const uint32_t rows = (blocks + per - 1) / per, last = blocks - (rows - 1) * per;
                for (bool xcd : {false, true}) {
                    std::vector<int> taken(rows * units, 0);
                    long work[8] = {};
                    for (uint32_t i = 0; i < rows * units; ++i) {
                        const mmm_a_place at = mmm_place_of_a(i, units, mmm_make_divisor(units), xcd);
                        if (at.down >= rows || at.unit >= units) { ++bad; continue; }
                        ++taken[at.down * units + at.unit];
                        work[i & 7u] += at.down == rows - 1 ? last : per;
                    }
                    for (int t : taken) bad += t != 1;
                    for (long w : work)
                        for (long v : work) bad += w - v > (long)per;   // XCDs differ by one workgroup
                }
            }
    std::printf("%d\n", bad);
    return 0;
}
"""


def _printed(tmp_path, text):
    source, program = tmp_path / "launch.cpp", tmp_path / "launch"
    source.write_text(text)
    subprocess.run([HIPCC, "-std=c++17", "--offload-host-only", "-x", "hip", "-I", CSRC, "-I", os.path.join(CSRC, "..", "..", "include"), str(source), "-x", "none",
                    mm.LIB_PATH, f"-Wl,-rpath,{os.path.dirname(mm.LIB_PATH)}", "-o", str(program)], check=True)
    done = subprocess.run([str(program)], capture_output=True, text=True, timeout=60)
    assert done.returncode == 0, (done.returncode, done.stdout, done.stderr)
    return done.stdout.strip()


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no compiler")
def test_more_workgroups_than_a_grid_holds(tmp_path):
    """Refused as an invalid value; numbers of tiles that are 0 in 32 bits are divided by nowhere."""
    assert _printed(tmp_path, PROGRAM) == "1"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no compiler")
def test_groups_that_a_wave_walks(tmp_path):
    """All of them exist, also those of a wave past the last column, whose first batch is asked for before it is known to be empty."""
    assert _printed(tmp_path, GROUPS) == "0 1"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no compiler")
def test_blocks_of_a_over_the_workgroups(tmp_path):
    """Every block once, and as many for each XCD, also where the last row of workgroups has fewer blocks than the others."""
    assert _printed(tmp_path, PLACES) == "0"
