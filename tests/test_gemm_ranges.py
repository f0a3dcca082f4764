"""The column arithmetic of the products on the host (CPU only): how the waves
of a workgroup walk a row, over every length that a call accepts, and the sizes
the library works out for rows of close to 2^32 columns."""
import os
import shutil
import subprocess

import pytest

from paper_2504_11651_amd import codec

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2504_11651_amd", "csrc")

WALK = r"""
#include <cstdio>
#include <cstdlib>
#include "df11_gemm_ranges.h"
using namespace df11gemm;
// every column of [0, end) once: wave w takes the ranges w, w + 4, ... in
// order, slab by slab, and each slab after the last of a range opens the next
int main(int argc, char **argv) {
    if (argc == 3) return least_ranges(static_cast<uint32_t>(strtoull(argv[2], nullptr, 10)));
    const uint64_t end = strtoull(argv[1], nullptr, 10);
    const uint32_t range = rows_range(static_cast<uint32_t>(end));
    if (range % kSlabCols || range > kRangeCols || range == 0) return 2;
    uint64_t covered = 0;
    for (uint32_t w = 0; w < kRowsWaves; ++w) {
        Slab s;
        uint64_t want = uint64_t{w} * range;
        bool any = first_slab(static_cast<uint32_t>(end), range, w, &s);
        if (any != (want < end)) return 3;
        while (any) {
            const uint64_t stop = want + range < end ? want + range : end;
            for (uint64_t k = want; k < stop; k += kSlabCols) {
                if (s.k0 != want || s.k1 != stop || s.k != k) return 4;
                const bool last = stop - k <= kSlabCols;
                if (last_of_range(s) != last) return 5;
                covered += last ? stop - k : kSlabCols;
                Slab n;
                any = next_slab(static_cast<uint32_t>(end), range, s, &n);
                if (!any && !(last && want + uint64_t{kRowsWaves} * range >= end)) return 6;
                if (any) s = n;
            }
            want += uint64_t{kRowsWaves} * range;
            if (any != (want < end)) return 7;
        }
    }
    return covered == end ? 0 : 8;
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("walk")
    (d / "walk.cpp").write_text(WALK)
    exe = str(d / "walk")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-Werror",
                    "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC,
                    str(d / "walk.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("cols", [64, 192, 256, 320, 1024, 1088, 1792, 1920, 4032, 4096, 4160, 14336,
                                  65536, 2 ** 31 - 8192, 2 ** 31 - 1088, 2 ** 31 - 64, 2 ** 31])
def test_waves_cover_every_column_once(walk, cols):
    """Up to the most columns a workgroup holds."""
    r = subprocess.run([walk, str(cols)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stderr)


@pytest.mark.parametrize("cols,parts", [(2 ** 31, 1), (2 ** 31 + 64, 2), (2 ** 32 - 64, 2)])
def test_longer_rows_are_split(walk, cols, parts):
    r = subprocess.run([walk, "split", str(cols)], capture_output=True, text=True, timeout=60)
    assert r.returncode == parts


@pytest.mark.parametrize("cols", [64, 4096, 14336, 2 ** 31, 2 ** 32 - 2048, 2 ** 32 - 1024,
                                  2 ** 32 - 64])
@pytest.mark.parametrize("tokens", [1, 8, 9, 16, 17, 64])
def test_workspace_of_long_rows(cols, tokens):
    """Partial sums of ranges of about 1024 columns up to 8 tokens, of half of
    4096 above, in whole slabs of 256; none where a row is one range."""
    ranges = -(-cols // 1024) if tokens <= 8 else 2 * -(-cols // 4096)
    kc = min(-(--(-cols // ranges) // 256) * 256, cols)
    parts = -(-cols // kc)
    want = 4 * 16 * parts * tokens if parts > 1 else 0
    assert codec.gemm_workspace_bytes([(0, 16, cols)], tokens) == want
