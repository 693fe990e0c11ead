"""The predictors' feature loads of partial tiles stay inside the feature array: a host program walks
the offsets of every lane for every tile height. A load that starts inside the tile's rows lies
inside them whole, any other starts at or past their end (where the hardware drops it), and the loads
inside bring every 16-byte unit of every row exactly once, to its place in LDS."""
import os
import subprocess

import paper_2606_12950_amd as M

CSRC = os.path.join(os.path.dirname(M.LIBRARY_PATH), "csrc")

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "feature_load.h"
using namespace maestro;

// offset(load, wave, lane) of a tile of `most` rows; swizzle: the unit that a lane's place holds
template <class Offset, class Place>
int walk(const char* form, int most, int loads, Offset offset, Place place) {
  for (int rows = 1; rows <= most; ++rows) {
    const unsigned size = rows * kFeatureRow;
    std::vector<int> seen(size / 16, -1);
    for (int l = 0; l < loads; ++l)
      for (int wave = 0; wave < 4; ++wave)
        for (int lane = 0; lane < 64; ++lane) {
          const unsigned o = offset(l, wave, lane);
          if (o % 16 != 0 || (o < size && o + 16 > size)) return std::printf("%s rows %d: offset %u\n", form, rows, o);
          if (o >= size) continue;
          if (seen[o / 16] != -1) return std::printf("%s rows %d: offset %u twice\n", form, rows, o);
          seen[o / 16] = place(l, wave, lane);
          const int row = o / kFeatureRow, unit = o % kFeatureRow / 16;
          const int want = loads == 32 && most == 256 ? row * 8 + ((unit & 7) ^ ((row >> 1) & 7)) + 256 * 8 * (unit >> 3)
                                                      : row * 32 + (unit ^ (row & 15));
          if (seen[o / 16] != want) return std::printf("%s rows %d: offset %u at %d\n", form, rows, o, seen[o / 16]);
        }
    for (int s : seen)
      if (s == -1) return std::printf("%s rows %d: a unit is not read\n", form, rows);
  }
  return 0;
}

int main() {
  int bad = 0;
  // place: 16-byte units from the buffer's start (1 KB a load, four wavefronts one after another)
  auto place = [](int l, int wave, int lane) { return (l * 4 + wave) * 64 + lane; };
  bad |= walk("split 32", 32, 4, [](int l, int w, int i) { return feature_offset_split(l, w, i); }, place);
  bad |= walk("split 64", 64, 8, [](int l, int w, int i) { return feature_offset_split(l, w, i); }, place);
  bad |= walk("rows", 128, 16, [](int l, int w, int i) { return feature_offset_rows(l / 8, l % 8, w, i); }, place);
  bad |= walk("slices", 256, 32, [](int l, int w, int i) { return feature_offset_slice(l / 8, l % 8, w, i); }, place);
  return bad ? 1 : 0;
}
"""


def test_no_feature_load_passes_the_end_of_a_partial_tile(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", f"-I{CSRC}", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_loads_that_may_pass_the_end_carry_no_scalar_offset():
    # the hardware compares the per-lane offset with the buffer's size; one more offset beside it is only
    # for loads inside their buffer (weights and biases)
    for name in ("predict.hip", "predict_split.hip"):
        text = open(os.path.join(CSRC, name)).read()
        for at in range(len(text)):
            if text.startswith("dma16(", at):
                assert text[at:].split("(")[1].split(",")[0] in ("r1", "rs_w2", "rs_w3", "rb1", "rb2", "l.rs"), text[at:at + 60]
        assert "feature_offset" in text and "dma16_once(rs, " in text
    header = open(os.path.join(CSRC, "mlp.h")).read()
    once = header.split("void dma16_once(")[1].split("}")[0]
    assert "buffer_load_dwordx4 %2, %3, 0 offen nt lds" in once
