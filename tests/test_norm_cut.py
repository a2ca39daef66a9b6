"""How a LayerNorm with the contraction behind it is cut for few rows (norm_cut, few_rows.h), without a GPU."""
import subprocess

import pytest

import test_gpu_norm_rows as G
from paper_2505_23317_amd import build

DRIVER = """
#include "few_rows.h"
#include <cstdio>
using namespace cfdetr;
int main() {
  for (int N : {384, 768, 1152, 1536, 1920, 2304, 2688, 3072, 4608})
    for (int rows = 1; rows <= 20000; rows += rows < 100 ? 1 : rows < 8000 ? 37 : 370)
      for (int cus : {256, 64}) {
        const NormCut c = norm_cut(rows, N, cus);
        std::printf("%d %d %d %d %d %d %d %d\\n", N, rows, cus, c.mt, c.mt ? c.shares : 0, c.mt ? c.per_share : 0,
                    c.mt ? c.group_bits : 0, c.mt ? norm_units(rows, c.mt, c.shares, c.group_bits) : 0);
      }
  for (int N : {HIDDEN, 2304})
    for (int frames : {FRAMES, MOST}) {
      const NormCut c = norm_cut(CELLS * frames, N, 256);
      std::printf("gpu %d %d %d %d %d\\n", N, frames, c.mt, c.mt ? c.shares : 0, c.mt ? c.per_share : 0);
    }
  for (int N = 384; N <= 6144; N += 384)
    for (int rows = 1; rows <= 20000; rows += rows < 2000 ? 1 : 37)
      for (int cus : {256, 64, 304})
        for (int gelu = 0; gelu < 2; ++gelu)
          if (few_rows_tiles(rows, N, 768, gelu != 0, cus) && norm_cut(rows, N, cus).mt == 0)
            std::printf("apart %d %d %d %d\\n", N, rows, few_rows_tiles(rows, N, 768, gelu != 0, cus),
                        few_rows_cut(rows, N, 768, 1, cus).most <= cus / 8);
  for (int rows = 1; rows <= 6000; ++rows)
    for (int cus : {256, 64}) std::printf("ahead %d %d %d\\n", rows, cus, norm_reads_ahead(rows, cus));
}
"""


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    at = tmp_path_factory.mktemp("cut")
    sizes = {"HIDDEN": G.HIDDEN, "FRAMES": G.FRAMES, "MOST": (G.MOST,), "CELLS": (G.CELLS[0] * G.CELLS[1],)}
    text = DRIVER
    for name, values in sizes.items():
        text = text.replace(name, ", ".join(map(str, values)))
    (at / "driver.hip").write_text(text)
    r = subprocess.run([build._hipcc(), "--offload-arch=gfx950", "-std=c++17", "-I", build.CSRC, str(at / "driver.hip"), "-o",
                        str(at / "driver")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    out = subprocess.run([str(at / "driver")], capture_output=True, text=True, check=True).stdout
    return [line.split() for line in out.splitlines()]


@pytest.fixture(scope="module")
def cuts(lines):
    return [tuple(map(int, line)) for line in lines if line[0].isdigit()]


def test_every_tile_and_strip_once_and_a_workgroup_a_cu(cuts):
    """The kernel's way from a workgroup to its units: XCD x has an equal run of the units of its group of shares."""
    seen = set()
    for N, rows, cus, mt, shares, per, bits, most in cuts:
        if mt == 0:
            seen.add(0)
            continue
        strips, tiles, xcds = N // 32, -(-rows // (32 * mt)), 8 >> bits
        assert shares * per >= strips > (shares - 1) * per and per <= 32
        assert most <= cus // 8
        got = []
        for xcd in range(8):
            group, nth = xcd >> (3 - bits), xcd & (xcds - 1)
            first = (shares * group) >> bits
            n = ((shares * (group + 1)) >> bits) - first
            lo, hi = (tiles * n * nth) >> (3 - bits), (tiles * n * (nth + 1)) >> (3 - bits)
            assert hi - lo <= most
            got += [(u // n, first + u % n) for u in range(lo, hi)]
        assert sorted(got) == [(t, s) for t in range(tiles) for s in range(shares)]
        seen.add(mt)
    assert seen == {0, 1, 2}


@pytest.mark.parametrize("N, rows, mt", [(2304, 1300, 1), (3072, 1300, 1), (3072, 2600, 2), (2304, 5200, 2), (3072, 5200, 2),
                                         (2304, 8200, 0), (3072, 16063, 0), (384, 4000, 1), (384, 16300, 2), (768, 4000, 1),
                                         (768, 16300, 2), (1152, 8100, 2), (1920, 8100, 2), (1920, 9600, 0), (4608, 2400, 2)])
def test_by_the_figures(cuts, N, rows, mt):
    """Heights at the row counts that the comments at norm_cut and its kernel have figures for (the nearest below)."""
    at = max((r for n, r, cus, *_ in cuts if n == N and cus == 256 and r <= rows))
    assert [c[3] for c in cuts if c[:3] == (N, at, 256)] == [mt]


# rows up to which a pass is faster with two launches, and from which with one (one context over and over or three in turn)
@pytest.mark.parametrize("N, two, one", [(768, 900, 1500), (1152, 612, 918), (1536, 612, 720), (2304, 324, 400), (3072, 288, 330),
                                         (4608, 64, 210)])
def test_fewest_rows_by_the_figures(cuts, N, two, one):
    for n, rows, cus, mt, *_ in cuts:
        if n == N and cus == 256 and (rows <= two or one <= rows <= 2 * one):
            assert (mt == 0) == (rows <= two), rows


def test_as_few_strips_as_wavefronts(cuts):
    """No share has more rounds of eight strips than its width needs: N = 1152 at 1,000 rows is five shares of eight strips
    at most and not four of nine, which would be two rounds."""
    at = {(n, rows): (shares, per) for n, rows, cus, mt, shares, per, *_ in cuts if cus == 256 and mt}
    near = min((r for n, r in at if n == 1152 and r >= 1000))
    assert at[1152, near] == (5, 8)


def test_weights_are_asked_for_ahead_by_the_figures(lines):
    """Rows at which a pass is slower, and faster, with the weights behind an attention launch asked for during it."""
    on = {int(rows): got == "1" for k, rows, cus, got, *_ in (v for v in lines if v[0] == "ahead") if cus == "256"}
    assert not any(on[rows] for rows in (400, 576, 600))
    assert all(on[rows] for rows in (720, 900, 1200, 2000, 4800, 5200))


def test_few_row_kernel_only_with_a_workgroup_a_cu(lines):
    """What follows a LayerNorm of width 768 in a launch of its own for few rows takes 32 rows a workgroup, one a CU: the
    figures at few_rows_tiles name no other form for it."""
    apart = [tuple(map(int, v[1:])) for v in lines if v[0] == "apart"]
    assert {n for n, *_ in apart} == set(range(384, 6145, 384))
    assert all(tiles == 1 and alone for _, _, tiles, alone in apart)


def test_what_the_gpu_test_covers(lines):
    """The batches of test_gpu_norm_rows.py: every one has a launch of the kind under test (the largest at the
    narrower hidden widths), at both heights and in two to twelve shares, even ones and uneven ones; the batch that they
    are compared with has none."""
    cut = {(int(n), int(f)): tuple(map(int, rest)) for k, n, f, *rest in (v for v in lines if v[0] == "gpu")}
    for ffn in G.HIDDEN:
        assert cut[ffn, G.MOST][0] == cut[2304, G.MOST][0] == 0
        assert all(cut[ffn, f][0] or cut[2304, f][0] for f in G.FRAMES if f <= 40 or ffn < 2304)
        assert {cut[ffn, f][0] for f in G.FRAMES} >= {1, 2}
    shares = {c[1] for c in cut.values() if c[0]}
    assert min(shares) == 2 and max(shares) == 12
    assert any(shares * per != ffn // 32 for ffn in G.HIDDEN[1:] for mt, shares, per in (cut[ffn, f] for f in G.FRAMES) if mt)
