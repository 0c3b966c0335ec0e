"""Index rules of the grid kernels, compiled for the host from the kernels' own header."""
import subprocess
from pathlib import Path

ROOT = Path(__file__).resolve().parent.parent

PROGRAM = r"""
#include <cstdio>
#include "scpic_internal.h"
int main()
{
    for (int pipe = 0; pipe < 2; ++pipe)
        for (int nx = 8; nx <= 256; nx += pipe ? nx : 1) {
            int mx = 1;
            while (mx < 2 * nx) mx *= 2;
            // the column kernels' lanes cover kMaxFft entries whatever mx is
            for (int k = 0; k < scpic::kMaxFft; ++k) {
                const int src = scpic::column_source(k, nx, mx, pipe != 0);
                int want = -1;
                if (k < nx) want = k;
                if (pipe && (k == 0 || k == nx)) want = -1;
                if (pipe && k > nx && k < mx) want = mx - k;
                if (src != want || src >= nx) {
                    std::printf("pipe %d nx %d mx %d k %d: %d, not %d\n", pipe, nx, mx, k, src, want);
                    return 1;
                }
            }
        }
    return 0;
}
"""


def test_column_entries_read_only_rows_of_the_spectrum(tmp_path):
    """Every lane of a column, those beyond its length among them, reads a row
    in [0, nx) or nothing (open boundary and grounded pipe)."""
    src, exe = tmp_path / "index.cpp", tmp_path / "index"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    f"-I{ROOT / 'include'}", f"-I{ROOT / 'paper_2010_11540_amd' / 'csrc'}",
                    str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
