"""Entries of empty cells of the traversal index (no GPU needed): the box an
entry names lies inside the empty box it was made from and holds the whole
octree cube of its cell, at every size of grid and cube, so that a walk never
takes more steps through empty space than the octree's own cells are."""
import subprocess

from paper_2103_14024_amd import _build

SRC = r"""
#include <hip/hip_runtime_api.h>
#include <cstdio>
#include <cstdlib>
#include "po_internal.h"
int main() {
    std::srand(1);
    long n = 0;
    for (int D = 4; D <= PO_MAX_DEPTH; ++D) {
        const int G = D - 3 < kIdxMaxGrid ? D - 3 : kIdxMaxGrid, unit = D - G, N = 1 << G;
        for (int up = 0; up < G; ++up)
            for (int rep = 0; rep < 2000; ++rep) {
                int c[3], lo[3], hi[3];
                for (int k = 0; k < 3; ++k) {
                    c[k] = std::rand() % N;
                    lo[k] = c[k] >> up << up;
                    hi[k] = lo[k] + (1 << up) - 1;
                    lo[k] -= std::rand() % 16;
                    hi[k] += std::rand() % 16;
                    if (lo[k] < 0) lo[k] = 0;
                    if (hi[k] >= N) hi[k] = N - 1;
                }
                const int32_t e = po_index_cube_entry(c, lo, hi, up, unit);
                const int u = po_index_unit(e), cube = po_index_cube(e);
                bool ok = e < 0 && u >= unit && cube == unit + up;
                for (int k = 0; k < 3; ++k) {  // in finest cells
                    const int at = c[k] << unit, below = e >> (8 * k) & 15, above = e >> (8 * k + 4) & 15;
                    const int a = ((at >> u) - below) << u, b = ((at >> u) + above + 1) << u;
                    const int ca = at >> cube << cube, cb = ca + (1 << cube);
                    ok = ok && a >= lo[k] << unit && b <= (hi[k] + 1) << unit && a <= ca && b >= cb;
                }
                if (!ok) {
                    std::printf("depth %d, up %d, cell %d %d %d: entry %08x\n", D, up, c[0], c[1], c[2], (unsigned)e);
                    return 1;
                }
                ++n;
            }
    }
    std::printf("%ld entries\n", n);
    return 0;
}
"""


def test_boxes_hold_the_cube(tmp_path):
    src, exe = tmp_path / "boxes.cpp", tmp_path / "boxes"
    src.write_text(SRC)
    subprocess.run([_build.hipcc(), "-std=c++17", "-I", _build.INCLUDE, "-I", _build.CSRC, str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
