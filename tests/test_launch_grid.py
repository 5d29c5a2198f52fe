"""Launch sizes of the set-up's kernels (csrc/grid.h): HIP refuses 2^32 threads
in a dimension; a device context takes up to 2^29 - 1 rows and 64 lanes a row."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = """
#include "grid.h"
int main()
{
    const int64_t top = (int64_t(1) << 29) - 1;
    for (int lanes : {1, 16, 64})
        for (int64_t n : {int64_t(1), int64_t(15), int64_t(16), int64_t(17), int64_t(1) << 20, (int64_t(1) << 26) - 1,
                          int64_t(1) << 26, int64_t(1) << 28, top}) {
            const int64_t blocks = amgiga::lanes_grid(n, lanes);
            if (blocks < 1 || blocks * 256 >= (int64_t(1) << 32)) return 1;
            // every row has its lanes in the first pass, or the grid strides
            if (blocks * 256 < n * lanes && blocks != amgiga::MAX_BLOCKS) return 2;
        }
    return int64_t(amgiga::MAX_BLOCKS) * 256 < (int64_t(1) << 32) ? 0 : 3;
}
"""


def test_grids_stay_below_the_launch_limit(tmp_path):
    src, exe = tmp_path / "grid.cpp", tmp_path / "grid"
    src.write_text(CODE)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2511_21268_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    subprocess.run([str(exe)], check=True)


def test_no_launch_of_the_set_up_multiplies_rows_by_lanes():
    """The kernels with several lanes a row and the slice fill take their grids
    from grid.h (fill pieces of 4M entries are small by themselves)."""
    with open(os.path.join(ROOT, "paper_2511_21268_amd", "csrc", "setup_dev.hip")) as f:
        text = f.read()
    assert "grid((n) *" not in text
    assert "dim3((unsigned)nslices)" not in text
