"""The rules of pdm_route.h (which kernels take the y and z passes), compiled
with g++ into a temporary directory, and the cases that tests put on the sweeps'
side of them."""
import ctypes
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_21552_amd", "csrc")
SHIM = """
#include "pdm_route.h"
extern "C" {
int sweep_fits(int n, int bx, int by, int bz) { return pdm::sweep_fits(n, bx, by, bz); }
int slice_y_wins(int n, int bx, int by, int bz) { return pdm::slice_y_wins(n, bx, by, bz); }
int row_lanes(int bx) { return pdm::row_lanes(bx); }
int batch_fits(const int* g, int count) { return pdm::batch_sweep_fits((const pdm::RouteGrid*)g, count); }
int volume_sweeps(const int* g) { return pdm::batch_volume_sweeps(*(const pdm::RouteGrid*)g); }
int parts(int bz) { return pdm::batch_sweep_parts(bz); }
int rows_class(int by) { return pdm::batch_sweep_class(by); }
}
"""


@functools.cache
def lib():
    with tempfile.TemporaryDirectory() as d:
        src, out = os.path.join(d, "r.cpp"), os.path.join(d, "r.so")
        with open(src, "w") as f:
            f.write(SHIM)
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, src, "-o", out], check=True)
        return ctypes.CDLL(out)


def sweep_fits(n, bx, by, bz):
    return bool(lib().sweep_fits(n, bx, by, bz))


def slice_y_wins(n, bx, by, bz):
    return bool(lib().slice_y_wins(n, bx, by, bz))


def _ints(grids):
    flat = [int(x) for g in grids for x in g]
    return (ctypes.c_int * len(flat))(*flat)


def batch_fits(grids):
    """grids: (n, Bx, By, Bz) of every volume."""
    return bool(lib().batch_fits(_ints(grids), len(grids)))


def volume_sweeps(grid):
    return bool(lib().volume_sweeps(_ints([grid])))


def bricks(shape, n):
    """(n, Bx, By, Bz) of a volume of [nz, ny, nx] voxels."""
    return (n,) + tuple((s + 3) // 4 for s in reversed(shape))


# One volume, (nz, ny, nx) and partitions: a map to a wave, two and four of
# them; whole quads and lanes, padded lanes, rows that end inside a quad; map
# counts that fill the last wave and that do not; an even and an odd number of
# planes; planes that are and are not whole blocks of rows; lines of over 256
# bricks.
SWEEP_CASES = [((795, 1024, 1024), 64), ((500, 1013, 1010), 64), ((512, 512, 512), 256), ((507, 509, 506), 253),
               ((1200, 512, 256), 255), ((1204, 510, 241), 254), ((1025, 504, 430), 255)]

# A batch of two large volumes and of small ones of every lane count, (nz, ny,
# nx) and partitions: both classes of row counts, planes cut in two parts and
# not, whole and ragged rows, map counts that fill a wave and that do not; among
# them volumes of narrow rows that keep the scans.
SWEEP_BATCH = [((800, 1000, 1010), 64), ((900, 1024, 1024), 61), ((36, 200, 400), 37), ((33, 197, 403), 37),
               ((60, 416, 256), 64), ((160, 80, 199), 33), ((7, 420, 217), 5), ((80, 8, 128), 64),
               ((600, 387, 123), 63), ((480, 380, 128), 64), ((64, 128, 64), 64), ((90, 70, 51), 7), ((100, 100, 27), 9),
               ((40, 50, 14), 64), ((61, 33, 9), 3)]
