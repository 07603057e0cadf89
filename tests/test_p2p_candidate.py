"""The near field's candidate rule (csrc/internal.h, p2p_candidate), compiled for the host: a source
without a position is no candidate, whatever the sign of its NaN.  (The distance from the targets' bounding
box passes over a NaN, and the sign bit that the cutoff test on the matrix cores reads in place of a
comparison is the NaN's.)"""
import os
import subprocess

from paper_2606_19059_amd import build as B

SRC = r"""
#include "internal.h"
#include <cmath>
#include <cstdio>
int main()
{
    const double nan = std::nan(""), rc2 = 0.04;
    // the box of one target at the origin, sources at (x, 0.1, 0)
    auto candidate = [&](double x) {
        const double d = std::fmax(0.0, std::fmax(-x, x));
        return (int)ewald::p2p_candidate(d * d + 0.01, x * x + 0.01, rc2);
    };
    std::printf("%d%d%d%d%d\n", candidate(0.1), candidate(0.0), candidate(0.2), candidate(nan), candidate(-nan));
    return 0;
}
"""


def test_a_source_without_a_position_is_no_candidate(tmp_path):
    src, exe = tmp_path / "t.hip", tmp_path / "t"
    src.write_text(SRC)
    cmd = [B._hipcc(), "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-I", B.CSRC, "-I",
           os.path.join(B.HERE, "..", "include"), str(src), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    assert subprocess.check_output([str(exe)], text=True).strip() == "11000"
