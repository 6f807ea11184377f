"""Which bytes the loads of consecutive rows into LDS touch (csrc/row_window.h), on the CPU: the arithmetic for every length, and that the
compiled kernels of attn_single.hip leave nothing to the bounds check that the hardware does not compare."""
import os
import re
import subprocess

from paper_2407_08454_amd import build as kbuild

CHECK = r"""
#include <cstdio>
#include "row_window.h"
using namespace kvm;
// One tile of `keys` rows from row0, 16 rows a window, as the kernel issues it.  A lane whose offset is below the window's size reads
// memory, the others get zeros.
static bool tile(int n, int row0, int keys, int chunks) {
    const int row_bytes = chunks * 16;
    for (int h = 0; h < keys / 16; ++h) {
        const RowWindow w = row_window(n, row0 + 16 * h, row_bytes);
        if (w.begin < 0 || w.bytes < 0 || w.begin + w.bytes != n * row_bytes) return false;
        for (int i = 0; i < 16 * chunks / 64; ++i)
            for (int lane = 0; lane < 64; ++lane) {
                const int in = row_of_lane(i, lane, chunks), off = in * row_bytes + offset_in_row(in, lane, chunks);
                const int row = row0 + 16 * h + in, slot = i * 64 + lane;
                if ((off < w.bytes) != (row < n)) return false;
                if (off >= w.bytes) continue;
                const int chunk = (slot % chunks) ^ (in & 15);     // what the kernel's fragment reads expect in this slot
                if (slot / chunks != in || w.begin + off != row * row_bytes + chunk * 16) return false;
                if (w.begin + off + 16 > n * row_bytes) return false;
            }
    }
    return true;
}
int main() {
    for (int n = 1; n <= 4096; ++n)
        for (int half = 0; half < 2; ++half) {
            const int keys = half ? 32 : 16, chunks = half ? 16 : 32;
            if (half && n > 2048) continue;
            for (int t = 0; t * keys < n; ++t)                     // (every tile of the shorter lengths, the last ones of all)
                if ((n <= 128 || (t + 3) * keys > n) && !tile(n, t * keys, keys, chunks)) { printf("n %d tile %d of %d\n", n, t, keys); return 1; }
        }
    return 0;
}
"""


def test_windows_of_rows_stay_inside_the_matrix(tmp_path):
    src, exe = tmp_path / "rows.cpp", tmp_path / "rows"
    src.write_text(CHECK)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", kbuild.CSRC, str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout


def test_buffer_loads_carry_no_scalar_offset(tmp_path):
    """The range check of a buffer load compares the lane's offset: a row in the scalar offset would be outside of it."""
    out = tmp_path / "single.s"
    flags = [f for f in kbuild.HIPCC_FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags + ["-I", kbuild.INCLUDE, "-I", kbuild.CSRC, "-S",
                   "--cuda-device-only", os.path.join(kbuild.CSRC, "attn_single.hip"), "-o", str(out)], check=True, capture_output=True)
    loads = re.findall(r"buffer_load_\w+ v\d+, s\[\d+:\d+\], (\S+) offen(.*) lds", out.read_text())
    assert len(loads) > 100
    assert {l[0] for l in loads} == {"0"}
    assert {l[1].strip() for l in loads} == {""}, "an offset in the instruction"
