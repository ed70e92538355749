"""Global cell indices of the step kernels' tiles on the host (hipcc only, no
GPU): a tile that takes the inner form computes them with a 24-bit product,
which must equal the plain 64-bit one in every grid that a handle accepts --
for every compiled tile shape, up to the widest grid its tile list can name."""
import os
import shutil
import subprocess

import pytest

from paper_1705_00614_amd import build

SOURCE = r"""
#include "%s"
#include <cstdio>

static long long bad = 0, inner = 0;

// first, second, middle and last columns of tiles, every row of tiles
template <int TX, int TY> void check(long long nx, long long ny) {
    const long long ntx = (nx + TX - 1) / TX, nty = (ny + TY - 1) / TY;
    if (ntx * nty >= (1LL << swe::TILE_BITS) || nx * ny > (1LL << 31) - 1) return;   // not accepted
    const long long cols[] = {0, 1, 5, ntx / 2, ntx - 3, ntx - 2, ntx - 1};
    for (long long tj = 0; tj < nty && tj < 6; ++tj)
        for (long long ti : cols) {
            if (ti < 0 || ti >= ntx) continue;
            const int tx0 = (int)(ti * TX), ty0 = (int)(tj * TY);
            if (swe::edge_tile<TX, TY>(tx0, ty0, (int)nx, (int)ny)) continue;
            ++inner;
            const int org = (ty0 - swe::HALO) * (int)nx + tx0;
            for (int y = -swe::HALO; y < TY + swe::HALO; ++y)
                for (int x : {-swe::HALO, 0, TX - 1, TX + swe::HALO - 1})
                    if (swe::inner_cell(org, x, y, (int)nx) != (ty0 + y) * nx + tx0 + x && ++bad < 4)
                        printf("tile %%dx%%d grid %%lld x %%lld at (%%d, %%d): cell (%%d, %%d)\n", TX, TY, nx, ny, tx0,
                               ty0, x, y);
        }
}

template <int TX, int TY> void shapes() {
    const long long wide[] = {1 << 24, 20000000, ((1LL << swe::TILE_BITS) - 1) / 3 * TX};
    for (long long ny : {2 * TY + swe::HALO, 3 * TY, 2 * TY + 8, 100, 4096})
        for (long long nx : {100LL, 777LL, 4096LL, 65537LL})
            check<TX, TY>(nx, ny);
    for (long long w : wide)
        for (long long nx : {w - 1, w, w + 1})
            for (long long ny : {2 * TY + swe::HALO, 2 * TY + 8, 3 * TY}) check<TX, TY>(nx, ny);
}

int main() {
    shapes<32, 32>();
    shapes<64, 16>();
    shapes<16, 16>();
    shapes<32, 16>();
    printf("%%lld inner tiles, %%lld wrong cells\n", inner, bad);
    return bad != 0 || inner == 0;
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_inner_tiles_index_every_accepted_grid(tmp_path):
    src, exe = tmp_path / "index.hip", tmp_path / "index"
    src.write_text(SOURCE % os.path.join(build.CSRC, "swe_step.hpp"))
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run(["hipcc"] + flags + ["-o", str(exe), str(src)], check=True, capture_output=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
