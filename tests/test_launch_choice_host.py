"""Into how many strips or runs the projection kernels cut their work, and the order of the weight gradient's tiles.  They
are compiled here into a small host program that deals the work items out as the card does - workgroups to the eight XCDs in
turn, on each to the compute unit that is free first - and compares the time of the choice with that of plain alternatives,
and the tiles of the fullest XCD with an even share."""

import os
import subprocess

import pytest

from paper_2605_17862_amd import build as b
from projection_cases import STRIPS_OF_SEVERAL_TILES

SOURCE = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "fopd_gemm.hip"
using namespace fopd;

CASES

// Steps until all items are done; an item of strip / run r takes length(r) and `start`, an empty workgroup nothing.
template <typename Length>
static double makespan(int tiles_m, int tiles_n, int runs, double start, Length length) {
  static double busy[8][32];
  for (auto& x : busy) for (double& c : x) c = 0.0;
  const int per = static_cast<int>(tile_groups(tiles_m, tiles_n));
  double last = 0.0;
  for (int g = 0; g < per * runs; ++g)
    for (int slot = 0; slot < 32; ++slot) {
      const TilePlace at = tile_place<true>(static_cast<unsigned>(g % per), static_cast<unsigned>(slot), tiles_m, tiles_n);
      if (at.m >= tiles_m || at.n >= tiles_n) continue;
      double* cu = std::min_element(busy[g % 8], busy[g % 8] + 32);
      *cu += length(at.m, g / per) + start;
      last = std::max(last, *cu);
    }
  return last;
}

// Every tile of every run comes once, whether a launch has a workgroup for each place or 256 that walk, and the same ones.
template <bool N_FIRST, bool WALK>
static bool walked(int tiles_m, int tiles_n, int steps, int splits) {
  {
    const unsigned grid = gemm_grid((splits * tile_groups(tiles_m, tiles_n) + 7) / 8, WALK);
    std::vector<int> seen(static_cast<size_t>(tiles_m) * tiles_n * splits, 0);
    for (unsigned block = 0; block < grid; ++block) {
      TileWalk<N_FIRST, WALK> walk = {tiles_m, tiles_n, steps, splits};
      GemmTile t;
      if (!walk.first(t, block)) continue;
      do {
        if (t.m0 < 0 || t.m0 % 256 || t.m0 / 256 >= tiles_m || t.n0 < 0 || t.n0 % 256 || t.n0 / 256 >= tiles_n) return false;
        if (t.split < 0 || t.split >= splits || t.steps < 1 || t.first != steps * t.split / splits ||
            t.first + t.steps != steps * (t.split + 1) / splits)
          return false;
        ++seen[(static_cast<size_t>(t.split) * tiles_n + t.n0 / 256) * tiles_m + t.m0 / 256];
      } while (walk.next(t));
      const GemmTile last = t;
      if (walk.next(t) || t.m0 != last.m0 || t.n0 != last.n0) return false;
    }
    for (int c : seen) if (c != 1) return false;
  }
  return true;
}

int main() {
  for (int tokens = 1; tokens <= 72; ++tokens)
    for (int vocab : {63, 125, 594, 1024}) {
      const int most = kLmStrips + kLmPairsExtra / (tokens * kLmTile);
      auto time = [&](int strips) {
        return makespan(strips, tokens, 1, 0.15, [&](int m, int) {
          return double((m + 1) * (long)vocab / strips - m * (long)vocab / strips);
        });
      };
      const int own = lm_strips(tokens, vocab);
      double plain = 1e30;
      for (int c : {8, 16, 32}) if (c <= most) plain = std::min(plain, time(c));
      std::printf("strips %d %d %d %d %.3f %.3f\n", tokens, vocab, own, most, time(own), plain);
    }
  for (int rows = 1; rows <= 32; ++rows)
    for (int cols : {4, 8, 10, 16, 20})
      for (int steps : {500, 2374}) {
        auto time = [&](int runs) {
          return makespan(cols, rows, runs, 13.0 / 1.6, [&](int, int r) {
            return double((r + 1) * (long)steps / runs - r * (long)steps / runs);
          });
        };
        const int most = std::min(steps * 64 / (cols * 256), 32);
        const int own = gemm_splits(cols * 256, rows * 256, steps * 64L, most);
        double plain = 1e30;
        for (int c : {1, 2, 4}) if (c <= most) plain = std::min(plain, time(c));
        std::printf("runs %d %d %d %d %.3f %.3f\n", rows * 1000 + cols, steps, own, most, time(own), plain);
      }
  for (int hidden = 1; hidden <= 40; ++hidden)
    for (int vocab : {3, 63, 125, 594, 1024}) {
      int tiles[8] = {}, seen = 0, most = 0;
      static bool once[64][1024];
      for (auto& x : once) for (bool& y : x) y = false;
      for (int g = 0; g < tile_groups(hidden, vocab); ++g)
        for (int slot = 0; slot < 32; ++slot) {
          const TilePlace at = tile_place<false>(static_cast<unsigned>(g), static_cast<unsigned>(slot), hidden, vocab);
          if (at.m >= hidden || at.n >= vocab) continue;
          if (at.m < 0 || at.n < 0 || once[at.m][at.n]) return 1;
          once[at.m][at.n] = true;
          ++seen;
          most = std::max(most, ++tiles[g % 8]);
        }
      std::printf("order %d %d %d %d\n", hidden, vocab, seen, most);
    }
  for (int T = 1; T <= 4200; T += T < 1400 ? 1 : 7)
    for (int V : {100, 385, 20001, 32000, 151936}) {
      const LmSplit s = lm_split(T, V);
      const long tiles = (T + 255) / 256, room = 32 * tiles * 256 + kLmPairsExtra;
      const long pairs = s.wide() ? (long)s.strips * T : (long)s.strips * s.whole * 256 + (long)s.tail_strips * 128;
      const long covered = s.wide() ? 384 : s.whole * 256L + (s.tail_strips > 0 ? 128 : 0);
      std::printf("split %d %d %d %ld %ld %ld %d\n", T, V, s.wide() || s.whole > 0 ? s.strips : s.tail_strips, room, pairs, covered,
                  (int)(s.wide() ? s.strips <= (V + 127) / 128 : 1));
    }
  for (const auto& c : kCases) {
    const LmSplit s = lm_split(c[0], c[1]);
    std::printf("case %d %d %d %d %d %d %d\n", c[0], c[1], (int)s.wide(), s.whole, s.strips, s.tail_strips,
                (c[1] + (s.wide() ? 127 : 255)) / (s.wide() ? 128 : 256));
  }
  for (int m : {1, 2, 4, 7, 8, 9, 16, 33, 594})
    for (int n : {1, 2, 3, 4, 5, 8, 64, 594})
      for (int splits : {1, 3, 8})
        for (int first : {0, 1}) {
          if (first ? !walked<true, true>(m, n, 19, splits) || !walked<true, false>(m, n, 19, splits)
                    : !walked<false, true>(m, n, 19, splits) || !walked<false, false>(m, n, 19, splits))
            return 2;
          std::printf("walk %d %d %d %d\n", m, n, splits, first);
        }
  for (int tiles : {1, 16, 125, 256, 257, 594, 9504})
    for (int steps : {1, 2, 64, 128, 129, 2374})
      for (int accumulate : {0, 1})
        std::printf("walks %d %d %d %d\n", tiles, steps, accumulate, static_cast<int>(gemm_walks(tiles, steps, accumulate != 0)));
}
"""


@pytest.fixture(scope="module")
def choices(tmp_path_factory):
    d = tmp_path_factory.mktemp("launch_choice")
    cases = ", ".join("{%d, %d}" % c[:2] for c in STRIPS_OF_SEVERAL_TILES)
    (d / "choice.hip").write_text(SOURCE.replace("CASES", "static const int kCases[][2] = {%s};" % cases))
    flags = [f for f in b.HIPCC_FLAGS if f not in ("-fPIC", "-shared", "-O3")]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags +
                   ["-O1", "-I", os.path.join(b.ROOT, "include"), "-I", os.path.join(b.PKG, "csrc"),
                    str(d / "choice.hip"), "-o", str(d / "choice")], check=True, capture_output=True)
    out = subprocess.run([str(d / "choice")], check=True, capture_output=True, text=True).stdout
    return [l.split() for l in out.splitlines()]


@pytest.mark.parametrize("what", ["strips", "runs"])
def test_no_slower_than_plain_choices(choices, what):
    rows = [r for r in choices if r[0] == what]
    assert len(rows) > 200
    for _, where, size, own, most, time, plain in rows:
        assert 1 <= int(own) <= int(most), (where, size, own)
        # 8, 16 or 32 strips, 1, 2 or 4 runs; the rule counts whole rounds only, hence the few per cent
        assert float(time) <= 1.08 * float(plain), (what, where, size, own, time, plain)


def test_tiles_of_the_weight_gradient_are_spread_evenly(choices):
    rows = [[int(x) for x in r[1:]] for r in choices if r[0] == "order"]
    assert len(rows) == 200
    for hidden, vocab, seen, most in rows:
        assert seen == hidden * vocab                        # each tile once (the program checks that none comes twice)
        lines, line = -(-vocab // 4), -(-hidden // 8)
        # an even share, and a group of 32 for each place of a line in which one XCD can be ahead
        assert most <= hidden * vocab / 8 + 32 * min(line, lines), (hidden, vocab, most)


def test_walking_workgroups_take_every_tile_once(choices):
    assert sum(r[0] == "walk" for r in choices) == 9 * 8 * 3 * 2           # the program stops at one that does not


def test_strips_of_whole_narrow_and_wide_token_tiles(choices):
    rows = [[int(x) for x in r[1:]] for r in choices if r[0] == "split"]
    assert len(rows) > 5000
    for T, V, strips, room, pairs, covered, filled in rows:
        assert strips >= 1 and covered >= T and filled, (T, V)
        assert pairs <= room, (T, V)                         # the workspace has so many (reference, sum) pairs


def test_only_launches_with_more_tiles_than_workgroups_walk(choices):
    rows = [[int(x) for x in r[1:]] for r in choices if r[0] == "walks"]
    assert len(rows) == 7 * 6 * 2
    for tiles, steps, accumulate, walks in rows:
        # the walk's code costs a launch 4 - 6 us, for nothing where no workgroup has a second tile
        assert walks == (tiles > 256 and steps <= 128 and not (accumulate and steps == 1)), (tiles, steps, accumulate)


def test_cases_of_strips_with_several_vocabulary_tiles(choices):
    rows = {(int(r[1]), int(r[2])): [int(x) for x in r[3:]] for r in choices if r[0] == "case"}
    assert len(rows) == len(STRIPS_OF_SEVERAL_TILES)
    for T, V, form, whole_rows in STRIPS_OF_SEVERAL_TILES:
        wide, whole, strips, tail_strips, vocab_tiles = rows[T, V]
        assert form == ("one" if wide else "shared" if tail_strips == 0 else "own" if whole > 0 else "narrow"), (T, V)
        assert whole * 256 == whole_rows, (T, V)
        assert form != "shared" or 0 < T - 256 * (whole - 1) <= 128, (T, V)
        # some strip has two tiles or more, in the own strips of a last tile too
        assert all(vocab_tiles > n for n in (strips, tail_strips) if n > 0), (T, V)
