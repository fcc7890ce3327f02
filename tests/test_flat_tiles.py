"""The choice of flat tiles by a kernel that addresses a tile's words with 32-bit offsets (CPU): the
host functions of the library's own header, compiled into a small program."""
import os
import subprocess

import pytest

from paper_2507_11067_amd import _build

PROGRAM = r"""
#include <stdio.h>
#include "mms_internal.h"
int main() {
    int nx, ny, nz, r, nt;
    long long sy;
    while (scanf("%d %d %d %d %d %lld", &nx, &ny, &nz, &r, &nt, &sy) == 6) {
        mms::Geom g{};
        g.nx = nx; g.ny = ny; g.nz = nz; g.sy = sy; g.rows = -1;
        const bool flat = mms::flat_tile32(g, r, nt, 256, 8);
        printf("%d %d %d\n", (int)flat, g.rows, g.nty);
    }
}
"""


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    d = tmp_path_factory.mktemp("flat")
    (d / "main.hip").write_text(PROGRAM)
    subprocess.run([_build._hipcc(), "--offload-host-only", "-std=c++20", "-I" + _build.INCLUDE,
                    "-I" + _build.CSRC, str(d / "main.hip"), "-o", str(d / "main")], check=True,
                   capture_output=True)

    def run(cases):
        text = "\n".join(" ".join(map(str, c)) for c in cases)
        out = subprocess.run([str(d / "main")], input=text, check=True, capture_output=True, text=True)
        return [tuple(map(int, l.split())) for l in out.stdout.splitlines()]
    return run


def test_flat_tiles_stay_within_32_bit_offsets(choose):
    """A tile is flat only where its last word's offset from its origin, rows + 2r - 1 rows down
    and a row's words across, fits 32 bits; pitches that the wide tile of 8 rows takes and a
    flat one cannot are left to the wide tile."""
    cases = [(nx, ny, nz, r, 512, sy) for nx in (1, 4, 9, 47, 100, 112) for ny, nz in ((300, 300), (40000, 8))
             for r in (1, 2, 3, 4) for sy in (128, 4096, 2 ** 22, 2 ** 24, 31580644, 2 ** 25, 2 ** 26, 2 ** 27)]
    seen = set()
    for (nx, ny, nz, r, nt, sy), (flat, rows, nty) in zip(cases, choose(cases), strict=True):
        if flat:
            assert (rows + 2 * r) * sy < 2 ** 32 and rows * nty >= ny and rows * ((nx + 3) // 4) <= nt
        else:
            assert (128 + 2 * r + 1) * sy >= 2 ** 32 and rows == -1
        seen.add((sy, flat))
    assert {(128, 1), (4096, 1), (2 ** 22, 1), (2 ** 26, 0), (2 ** 27, 0)} <= seen
