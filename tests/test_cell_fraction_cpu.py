"""The pass's one-conversion cell index and fraction, compiled for the host from the kernels' own
header, against the deposit's definition i = floor(t), a = floor((t - i) 4096 + 0.5)."""
import subprocess
from pathlib import Path

ROOT = Path(__file__).resolve().parent.parent

PROGRAM = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include "scpic_internal.h"

static long bad = 0;
static void check(double t)
{
    if (!(t >= 0.0 && t < 511.0)) return;
    const double fi = std::floor(t);
    const int want_i = (int)fi, want_a = (int)std::floor((t - fi) * 4096.0 + 0.5);
    int i, a;
    scpic::cell_fraction(t, i, a);
    if (i != want_i || a != want_a) {
        if (++bad < 10) std::printf("t = %a: (%d, %d), not (%d, %d)\n", t, i, a, want_i, want_a);
    }
}

int main()
{
    // every edge of the rounding (multiples of 1/8192, where cells and
    // fractions change) with its neighbours in the last places
    for (int k = 0; k <= 511 * 8192; ++k) {
        double t = k / 8192.0;
        check(t);
        double up = t, down = t;
        for (int n = 0; n < 3; ++n) {
            up = std::nextafter(up, 1e9);
            down = std::nextafter(down, -1.0);
            check(up);
            check(down);
        }
    }
    // the one value below which u + 0.5 is not exact, its neighbours, zeros, the smallest
    check((0.5 - 0x1p-54) / 4096.0);
    check(0.0);
    check(-0.0);
    check(5e-324);
    // any bit pattern below 511
    uint64_t s = 88172645463325252ull;
    for (long n = 0; n < 20000000; ++n) {
        s ^= s << 13;
        s ^= s >> 7;
        s ^= s << 17;
        double t;
        const uint64_t bits = (s >> 12) | ((1023ull - (s % 60) + 9) << 52);
        std::memcpy(&t, &bits, 8);
        check(t);
    }
    return bad ? 1 : 0;
}
"""


def test_cell_fraction_equals_the_deposits_definition(tmp_path):
    src, exe = tmp_path / "cell.cpp", tmp_path / "cell"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", f"-I{ROOT / 'include'}",
                    f"-I{ROOT / 'paper_2010_11540_amd' / 'csrc'}", str(src), "-o", str(exe)],
                   check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
