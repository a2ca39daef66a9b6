"""Host side of the kernels' launchers, without a GPU: arguments that no kernel applies are refused; which kernel
contractions of few rows go to."""
import os
import subprocess

import pytest

from paper_2505_23317_amd import build

DRIVER = """
#include "few_rows.h"
#include <cstdio>
using namespace cfdetr;
int main() {
  for (int bf16 = 0; bf16 < 2; ++bf16)
    for (Epilogue epi : {Epilogue::kBias, Epilogue::kBiasGelu, Epilogue::kBiasRelu, Epilogue::kBiasResidual})
      if (!(bf16 && epi == Epilogue::kBias))
        std::printf("scale %d\\n", (int)launch_gemm(nullptr, nullptr, nullptr, 64, 64, epi, nullptr, nullptr, bf16 != 0, nullptr,
                                                   64, 64, nullptr, 0.5f));
  const int shapes[][3] = {SHAPES};
  for (const auto& n : shapes)
    for (int m = 1; m <= 12000; m += m % 10 == 0 ? 1 : 9)
      for (int cus : {256, 64}) {
        const FewCut one = few_rows_cut(m, n[0], n[1], 1, cus), two = few_rows_cut(m, n[0], n[1], 2, cus);
        std::printf("tiles %d %d %d %d %d %d %d %d\\n", n[0], n[1], n[2], m, cus, one.row_bits, two.row_bits,
                    few_rows_tiles(m, n[0], n[1], n[2] != 0, cus));
      }
  for (int d : {256, 384})
    for (int rows : {8192, 16384, 18432, 24576, 32768, 102400, 112896})
      std::printf("height %d %d %d\\n", d, rows, wide_layer_tiles(d, rows, 256));
  for (int project = 0; project < 2; ++project)
    for (int parts = 1; parts <= 16; ++parts)
      for (int tiles = 1; tiles <= 120; ++tiles) {
        std::printf("share %d %d %d %d", project, parts, tiles, parts_of_a_share(tiles, parts, 384, project != 0, 256));
        for (int n = 1; n <= parts; ++n) {
          const SlimBytes b = slim_bytes(384, n, project != 0);
          std::printf(" %d", few_rows_cut(tiles, (parts + n - 1) / n, b.row, b.part, b.tile, 256).row_bits);
        }
        std::printf("\\n");
      }
  for (int ffn : {384, 768, 1152, 1536, 1920})
    for (int m = 1; m <= 4000; m += m % 10 == 0 ? 1 : 9)
      for (int cus : {256, 64}) {
        const FewDown down = few_rows_down(m, 384, ffn, cus);
        std::printf("down %d %d %d %d %d %d\\n", ffn, m, cus, down.mt, down.waves,
                    few_rows_cut((m + 31) / 32, 6, 64.0 * ffn, 128.0 * ffn, 192.0 * ffn, cus).row_bits);
      }
}
"""
# N, K, GELU behind it
SHAPES = [(768, 768, 0), (768, 3072, 0), (2304, 768, 0), (3072, 768, 1), (1536, 768, 1), (768, 1536, 0), (384, 3072, 0),
          (2304, 384, 1), (1152, 384, 0)]


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    """What the driver prints; it calls only what ends before a launch, and sees no GPU."""
    objects = [os.path.join(build.HERE, "_build", s.replace(".hip", ".o")) for s in build.SOURCES]
    if not all(os.path.exists(o) for o in objects):
        pytest.skip("the library has not been built here")
    at = tmp_path_factory.mktemp("rules")
    (at / "driver.hip").write_text(DRIVER.replace("SHAPES", ", ".join("{%d, %d, %d}" % s for s in SHAPES)))
    hipcc = [build._hipcc(), "--offload-arch=gfx950"]
    for cmd in ([*hipcc, "-std=c++17", "-I", build.CSRC, "-c", str(at / "driver.hip"), "-o", str(at / "driver.o")],
                [*hipcc, str(at / "driver.o"), *objects, "-o", str(at / "driver")]):
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-3000:]
    got = subprocess.run([str(at / "driver")], capture_output=True, text=True, check=True,
                         env={**os.environ, "HIP_VISIBLE_DEVICES": "-1"}).stdout
    return [line.split() for line in got.splitlines()]


def test_a_factor_that_nothing_applies_is_refused(lines):
    """The activations, the residual form and the fp32 path have no factor: 1 is hipErrorInvalidValue."""
    assert [v for k, *v in lines if k == "scale"] == [["1"]] * 7


def _fullest(m, N, height, bits):
    """Tiles of the XCD with the most, as XcdTiles deals them: workgroup by workgroup."""
    tiles, parts, most = -(-m // height), N // 128, 0
    for xcd in range(8):
        rg, pg, part_bits = xcd & ((1 << bits) - 1), xcd >> bits, 3 - bits
        rows = ((tiles * (rg + 1)) >> bits) - ((tiles * rg) >> bits)
        most = max(most, rows * (((parts * (pg + 1)) >> part_bits) - ((parts * pg) >> part_bits)))
    return most


def test_few_rows_go_where_no_cu_gets_two(lines):
    """32 rows a workgroup, else 64, as long as no CU of any XCD gets a second workgroup; two only by the rules that
    the comment at few_rows_tiles has figures for."""
    seen = set()
    for k, *v in lines:
        if k != "tiles":
            continue
        N, K, gelu, m, cus, bits1, bits2, got = map(int, v)
        share = cus // 8
        one, two = _fullest(m, N, 32, bits1), _fullest(m, N, 64, bits2)
        want = 1 if one <= share else 2 if two <= share else 1 if one <= 2 * share else 0
        if want == 0 and two <= 2 * share and (gelu and N >= 2304 or N % 256 and K >= 2048 and 2 * two > 3 * share):
            want = 2
        assert got == want, (N, K, gelu, m, cus, one, two)
        seen.add((got, one <= share, two <= share))
    assert seen == {(1, True, True), (2, False, True), (1, False, False), (2, False, False), (0, False, False)}


def test_shares_of_a_row_tile(lines):
    """Of all splits of the parts the one that leaves the busiest CU the least, its columns and a start of 200."""
    for k, *v in lines:
        if k != "share":
            continue
        project, parts, tiles, got, *bits = map(int, v)
        cost = [-(-_fullest(32 * tiles, 128 * -(-parts // n), 32, bits[n - 1]) // 32) * (384 * project + 200 + 128 * n)
                for n in range(1, parts + 1)]
        assert cost[got - 1] == min(cost), (project, parts, tiles)


def test_second_matrix_of_few_rows(lines):
    """Width 384: 64 columns a workgroup where every one then has a CU of its own and K is whole rings of 48 blocks, else
    128, and 64 rows where 32 would give a CU two."""
    seen = set()
    for k, *v in lines:
        if k != "down":
            continue
        ffn, m, cus, mt, waves, bits = map(int, v)
        narrow = _fullest(m, 768, 32, bits) <= cus // 8   # (parts of 64 of 384 columns, as many as of 128 of 768)
        assert (waves == 2) == (narrow and ffn % 768 == 0), v
        assert waves == 4 or mt == 2 or 3 * -(-m // 32) <= cus, v
        assert waves == 4 or mt == 1, v
        seen.add((mt, waves))
    assert seen == {(1, 2), (1, 4), (2, 4)}


# rows at which one of the forms is the fastest by a tenth and more
@pytest.mark.parametrize("N, K, gelu, m, tiles", [
    (768, 3072, 0, 1300, 2), (768, 3072, 0, 2700, 0), (768, 768, 0, 2700, 0), (2304, 768, 0, 300, 1), (1152, 384, 0, 700, 1),
    (1152, 384, 0, 1420, 2), (2304, 384, 1, 1420, 2), (384, 3072, 0, 8500, 2), (384, 3072, 0, 10900, 0)])
def test_few_rows_by_the_figures(lines, N, K, gelu, m, tiles):
    assert ["tiles", *map(str, (N, K, gelu, m, 256))] + [str(tiles)] in [v[:6] + v[8:] for v in lines]


def test_rows_of_a_layer_workgroup_by_the_figures(lines):
    """The fastest of 32, 64 and 96 rows at the row counts that the comment at wide_layer_tiles has figures for."""
    got = {(int(d), int(rows)): int(mt) for k, *v in lines if k == "height" for d, rows, mt in [v]}
    want = {256: {8192: 1, 16384: 2, 24576: 3, 32768: 2, 102400: 2, 112896: 2},
            384: {8192: 1, 16384: 2, 18432: 3, 24576: 3, 32768: 2}}
    for d, heights in want.items():
        for rows, mt in heights.items():
            assert got[d, rows] == mt, (d, rows)
