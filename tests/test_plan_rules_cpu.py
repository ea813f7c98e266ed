"""The host rules that choose tiles (csrc/fb_plan_rules.hpp), compiled for the
host and evaluated without a GPU."""
import os
import subprocess

import pytest

from paper_2004_09883_amd import fb
from test_gpu_fft import BLOCK_Z_GRIDS, WIDE_X_GRIDS

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2004_09883_amd", "csrc")
LONG = [576, 648, 729, 768, 864, 972, 1024, 1152, 1296, 1458, 1536, 1728, 1944, 2048, 2187, 2304, 2592, 2916, 3072,
        3456, 3888, 4096]
WIDE_PROGRAM = r"""
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


# tiles of a contiguous pass and the wavefronts from which it moves them as blocks
BLOCK_PROGRAM = r"""
#include <cstdio>
#include "fb_plan_rules.hpp"
int main()
{
    using namespace fb;
    long n, np, es;
    int nt;
    while (scanf("%ld %ld %ld %d", &n, &np, &es, &nt) == 4) {
        const bool split = es == 16 && split_exchange((int)n), g = grouped((int)n, true, false);
        const GroupPlan gp = group_plan((int)n, g);
        const int p = pencils_per_wg((int)n, true, (int)es, false, split, g);
        const long tiles = (np + p - 1) / p, waves = tiles * ((p * gp.threads + 63) / 64);
        printf("%ld %ld %d\n", tiles, waves, block_waves((int)n, (int)es, gp.count == 1, nt != 0, false));
    }
}
"""


def compiled(d, program):
    """ask(rows of four integers) -> one tuple of integers per row"""
    (d / "rules.cpp").write_text(program)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(d / "rules.cpp"), "-o", str(d / "rules")], check=True)

    def ask(rows):
        r = subprocess.run([str(d / "rules")], input="\n".join("%d %d %d %d" % x for x in rows), capture_output=True,
                           text=True, check=True)
        return [tuple(map(int, line.split())) for line in r.stdout.split("\n") if line]
    return ask


@pytest.fixture(scope="module")
def wide(tmp_path_factory):
    """(n, pencils, inner, nt) -> (pencils per wide tile, wide or not)"""
    return compiled(tmp_path_factory.mktemp("wide"), WIDE_PROGRAM)


@pytest.fixture(scope="module")
def block(tmp_path_factory):
    """(n, pencils, element bytes, nt) -> (tiles, wavefronts, least wavefronts for blocks or 0)"""
    return compiled(tmp_path_factory.mktemp("block"), BLOCK_PROGRAM)


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


def test_blocks_need_several_wavefronts_per_cu(block):
    """No length moves blocks with fewer wavefronts than one per CU, or, with
    cached accesses, two."""
    for nt, floor in ((0, 512), (1, 256)):
        rows = [(n, 1, es, nt) for n in range(2, 512) for es in (8, 16)
                if n in (2 ** a * 3 ** b for a in range(10) for b in range(6))]
        assert all(least == 0 or least >= floor for _, _, least in block(rows))


def test_grids_of_the_gpu_test_move_as_blocks(block):
    """... and one plane of each does not."""
    for planes, want in ((None, True), (1, False)):
        rows = [(z, (planes or x) * y, 16 if dt == fb.FB_C128 else 8,
                 int((planes or x) * y * z * (16 if dt == fb.FB_C128 else 8) >= 192 << 20))
                for (x, y, z), dt in BLOCK_Z_GRIDS]
        for row, (_, waves, least) in zip(rows, block(rows)):
            assert (least > 0 and waves >= least) == want, (row, waves, least)


def test_groups_of_images_keep_their_pencils_in_32_bits(tmp_path):
    """Any number of images splits into groups whose pencils, a tile's
    overhang included, are numbered in 32 bits."""
    ask = compiled(tmp_path, r"""
#include <cstdio>
#include "fb_plan_rules.hpp"
int main()
{
    long side, b, c, d;
    while (scanf("%ld %ld %ld %ld", &side, &b, &c, &d) == 4)
        printf("%ld %ld\n", (long)fb::batch_images_per_group(side), (long)FB_MAX_PENCILS);
}
""")
    sides = [s for s in range(2, 4097) if s in {2 ** a * 3 ** b for a in range(13) for b in range(2)}]
    for side, (per, limit) in zip(sides, ask([(s, 0, 0, 0) for s in sides])):
        assert per >= 1 and per * side < limit <= 2 ** 32 - 2 ** 16
        # the largest batch the plan takes, 2^31 - 1 images, in the fewest groups
        assert -(-(2 ** 31 - 1) // per) <= -(-(2 ** 31 - 1) * side // (limit - 1)) + 1
