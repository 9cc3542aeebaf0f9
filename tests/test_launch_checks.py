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


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no compiler")
def test_more_workgroups_than_a_grid_holds(tmp_path):
    """Refused as an invalid value; numbers of tiles that are 0 in 32 bits are divided by nowhere."""
    source, program = tmp_path / "launch.cpp", tmp_path / "launch"
    source.write_text(PROGRAM)
    subprocess.run([HIPCC, "-std=c++17", "--offload-host-only", "-x", "hip", "-I", CSRC, "-I", os.path.join(CSRC, "..", "..", "include"), str(source), "-x", "none",
                    mm.LIB_PATH, f"-Wl,-rpath,{os.path.dirname(mm.LIB_PATH)}", "-o", str(program)], check=True)
    done = subprocess.run([str(program)], capture_output=True, text=True, timeout=60)
    assert done.returncode == 0 and done.stdout.strip() == "1", (done.returncode, done.stdout, done.stderr)
