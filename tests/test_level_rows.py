"""The rule by which the per-cube kernels stage a cube's row of partial sums in
LDS, up to rows of 2^31 and more values (255 trials of 2^34 points), evaluated
by the compiler: a signed overflow is no constant and fails the compilation."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = """
#include "zmc_kernels.hpp"
constexpr long kFit = zmc::kStage / zmc::kLevelThreads;
static_assert(zmc::row_fits(1) && zmc::row_fits(kFit) && !zmc::row_fits(kFit + 1), "the edge");
static_assert(!zmc::row_fits(1l << 22) && !zmc::row_fits(1l << 23) && !zmc::row_fits(1l << 24), "times 512 or 256");
static_assert(!zmc::row_fits((1l << 32) / zmc::kLevelThreads) && !zmc::row_fits((1l << 32) + 1), "wrapped to 0 and 1");
static_assert(!zmc::row_fits(255l << 26) && !zmc::row_fits(0x7FFFFFFFl), "the largest accepted rows");
"""


def test_rows_that_fit(tmp_path):
    sys.path.insert(0, ROOT)
    from paper_1902_07916_amd import build
    src = tmp_path / "rows.hip"
    src.write_text(SRC)
    subprocess.run([build.hipcc(), "--offload-host-only", "-std=c++17", "-fsyntax-only", "-I" + build.CSRC,
                    "-I" + build.INCLUDE, str(src)], check=True)
