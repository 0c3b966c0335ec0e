"""The automatic choice of a pass's workgroup size, compiled for the host from the kernels' own header."""
import subprocess
from pathlib import Path

ROOT = Path(__file__).resolve().parent.parent

PROGRAM = r"""
#include <cstdio>
#include "scpic_internal.h"
static int bad = 0;
static void want(long long n, int limit, int cu, int threads)
{
    const int got = scpic::automatic_pass_threads(n, limit, cu);
    if (got != threads) {
        ++bad;
        std::printf("n %lld, %d workgroups, %d units: %d, not %d\n", n, limit, cu, got, threads);
    }
}
int main()
{
    // a beam of more than one round of 512 threads per workgroup takes 1024, whatever bounds the workgroups
    for (int cu : {1, 64, 256})
        for (int limit : {1, 2, 16, 64, 256, 512}) {
            const long long round = 512ll * (limit < cu ? limit : cu);
            for (long long n : {round + 1, round + 511, 2 * round, 100 * round})
                want(n, limit, cu, 1024);
            want(round, limit, cu, 512);
            want(1, limit, cu, 512);
        }
    // a caller's limit of two workgroups
    want(60001, 2, 256, 1024);
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
