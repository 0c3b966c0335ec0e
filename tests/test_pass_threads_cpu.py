"""The automatic choice of a pass's workgroup size, compiled for the host from the kernels' own header."""
import subprocess
from pathlib import Path

ROOT = Path(__file__).resolve().parent.parent

PROGRAM = r"""
#include <cstdio>
#include "scpic_internal.h"
static int bad = 0;
static void want(long long n, long long cells, int limit, int cu, int threads)
{
    const int got = scpic::automatic_pass_threads(n, cells, limit, cu);
    if (got != threads) {
        ++bad;
        std::printf("n %lld, %lld nodes, %d workgroups, %d units: %d, not %d\n", n, cells, limit, cu, got,
                    threads);
    }
}
int main()
{
    // a beam of more than one round of 512 threads per workgroup takes 1024, whatever bounds the workgroups
    for (int cu : {1, 64, 256})
        for (int limit : {1, 2, 16, 64, 256, 512})
            for (long long cells : {64ll, 4096ll, 10240ll, 10244ll, 65536ll}) {
                const long long round = 512ll * (limit < cu ? limit : cu);
                for (long long n : {round + 1, round + 511, 2 * round, 100 * round})
                    want(n, cells, limit, cu, 1024);
                want(round, cells, limit, cu, cells <= 10240 ? 512 : 1024);
                want(round / 2, cells, limit, cu, 512);
                want(1, cells, limit, cu, 512);
            }
    // a caller's limit of two workgroups
    want(60001, 128 * 128, 2, 256, 1024);
    // large grids from half the compute units on
    want(131072, 256 * 256, 256, 256, 1024);
    want(100000, 200 * 200, 256, 256, 1024);
    want(131072, 64 * 64, 256, 256, 512);
    return bad ? 1 : 0;
}
"""


def test_small_beams_spread_only_while_no_workgroup_has_a_second_round(tmp_path):
    src, exe = tmp_path / "threads.cpp", tmp_path / "threads"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    f"-I{ROOT / 'include'}", f"-I{ROOT / 'paper_2010_11540_amd' / 'csrc'}",
                    str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
