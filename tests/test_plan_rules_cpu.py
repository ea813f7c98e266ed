"""The host rules that choose tiles (csrc/fb_plan_rules.hpp), compiled for the
host and evaluated without a GPU."""
import os
import subprocess

import pytest

from test_gpu_fft import WIDE_X_GRIDS

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2004_09883_amd", "csrc")
LONG = [576, 648, 729, 768, 864, 972, 1024, 1152, 1296, 1458, 1536, 1728, 1944, 2048, 2187, 2304, 2592, 2916, 3072,
        3456, 3888, 4096]
PROGRAM = r"""
#include <cstdio>
#include "fb_plan_rules.hpp"
int main()
{
    using namespace fb;
    long n, np, inner;
    int nt;
    while (scanf("%ld %ld %ld %d", &n, &np, &inner, &nt) == 4) {
        const int p = pencils_per_wg((int)n, false, 16, false, true, grouped((int)n, false, false));
        printf("%d %d\n", p, has_wide((int)n, false) && wide_pays((int)n, p, np, inner, nt != 0) ? 1 : 0);
    }
}
"""


@pytest.fixture(scope="module")
def wide(tmp_path_factory):
    """(n, pencils, inner, nt) rows -> (pencils per wide tile, wide or not)"""
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(d / "rules.cpp"), "-o", str(d / "rules")], check=True)

    def ask(rows):
        r = subprocess.run([str(d / "rules")], input="\n".join("%d %d %d %d" % x for x in rows), capture_output=True,
                           text=True, check=True)
        return [tuple(map(int, line.split())) for line in r.stdout.split("\n") if line]
    return ask


def test_wide_tiles_need_enough_tiles_for_the_device(wide):
    """With fewer than 128 wide tiles most CUs have none, cached or not."""
    rows = [(n, np, inner, nt) for n in LONG for np in (1, 16, 64, 243, 256, 500) for inner in (np, 8, 27)
            for nt in (0, 1)]
    for row, (pencils, is_wide) in zip(rows, wide(rows)):
        assert not (is_wide and (row[1] + pencils - 1) // pencils < 128), row


def test_wide_tiles_of_large_grids_with_whole_lines(wide):
    """384 MiB, rows of 4096 pencils and more: every length but the ones whose
    narrow rows of 64 bytes the caches join is wide."""
    rows = [(n, (384 << 20) // (16 * n) // 8 * 8, (384 << 20) // (16 * n) // 8 * 8, 1) for n in LONG]
    assert all(w for _, w in wide(rows))
    # cached grids of up to 1024 points, and rows that start inside a line there
    rows = [(n, 8192, 8192, 0) for n in LONG if n <= 1024] + [(n, 39366, 39366, 1) for n in LONG if n <= 1024]
    assert not any(w for _, w in wide(rows))


def test_grids_of_the_gpu_test_are_wide(wide):
    rows = [(n, ny * nz, ny * nz, int(16 * n * ny * nz >= 192 << 20)) for n, ny, nz in WIDE_X_GRIDS]
    for row, (_, is_wide) in zip(rows, wide(rows)):
        assert is_wide, row
    assert {r[0] for r in rows} == set(LONG)
    assert not any(w for _, w in wide([(n, 91, 91, 0) for n in LONG]))
