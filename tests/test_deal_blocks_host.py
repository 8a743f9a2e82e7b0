"""The deal of 32-token blocks to wavefronts (kernels.h: make_deal_of_blocks, blocks_of): every block to one wavefront, units of two or four blocks
only where every unit has a compute unit of its own; and the state passes' workgroups (deal_state_pass)."""
import os
import shutil
import subprocess

import pytest

from tests.test_deal_host import ROCM, ROOT

PROGRAM = r"""
#include "kernels.h"
#include <cstdio>
#include <vector>
using namespace linattn;
int main() {
  long bad = 0, units[9] = {};
  for (int BH : {1, 2, 3, 12, 50, 87, 128, 255, 256, 257, 300})
    for (int blocks : {1, 2, 3, 4, 5, 7, 8, 9, 10, 11, 31, 32, 33, 64, 129, 255, 512, 513, 1024, 1025})
      for (int waves : {8, 12})
        for (bool even : {false, true}) {
          const Split s = make_deal_of_blocks(BH, blocks, waves, {4, 2, 5, 240}, even);
          bad += s.blocks != 2 && s.blocks != 4 && s.blocks != waves;
          bad += s.blocks < waves && (s.G > kCUs || !s.share || split_rounds(s) != 1);
          if (s.blocks < 8) ++units[s.blocks];
          std::vector<unsigned char> seen((size_t)BH * blocks, 0);
          const dim3 grid = grid_of(s);
          for (int gy = 0; gy < (int)grid.y; ++gy)
            for (int gx = 0; gx < (int)grid.x; ++gx)
              for (Share sh = first_share(s, gx, gy); sh.there; sh = next_share(s, gx, sh))
                for (int w = 0; w < waves; ++w) {
                  const Blocks b = blocks_of(s, sh, w, blocks);
                  bad += b.end > blocks || b.stride < 1 || b.first < 0;
                  for (int i = b.first; i < b.end && i >= 0; i += b.stride) ++seen[(size_t)sh.bh * blocks + i];
                }
          for (unsigned char c : seen) bad += c != 1;
        }
  // the state passes: every tile once, partial slots within those of the even split, two heads to a workgroup only where that saves tiles
  long by_head = 0;
  for (int BH : {1, 2, 3, 5, 7, 12, 13, 24, 30, 40, 87, 127, 128, 129, 255, 256, 300})
    for (int tiles : {1, 2, 3, 5, 8, 16, 21, 22, 33, 64, 138, 157, 256, 591})
      for (int relu : {0, 1}) {
        Plan p{};
        p.BH = BH;
        p.kind = relu ? kPhiRelu : kPhiHedgehog;
        p.bf16_math = true;
        Split& s = p.split;
        s.ntile = tiles;
        s.T = (long long)BH * tiles;
        s.G = BH > kSlots ? BH : (int)(s.T < kSlots ? s.T : kSlots);
        finish_split(s);
        auto slots = [&] {
          int most = 1;
          for (long long bh = 0; bh < BH; ++bh) {
            const int cnt = split_owner(s, (bh + 1) * tiles - 1) - split_owner(s, bh * tiles) + 1;
            most = cnt > most ? cnt : most;
          }
          return most;
        };
        const int even_slots = s.PS = slots(), rounds = split_rounds(s), G = s.G;
        deal_state_pass(&p);
        by_head += s.G != G;
        bad += s.PS < slots() || s.PS > even_slots || split_rounds(s) > rounds + (rounds >= 4 && !relu);
        long long next = 0;
        for (int g = 0; g < s.G; ++g) {
          bad += split_lo(s, g) != next;
          next = split_lo(s, g + 1);
          bad += s.G != G && split_head(s, split_lo(s, g)) != split_head(s, next - 1);
        }
        bad += next != s.T;
      }
  bad += by_head == 0;
  printf("bad %ld two %ld four %ld\n", bad, units[2], units[4]);
  return bad != 0 || units[2] == 0 || units[4] == 0;
}
"""


EVEN = r"""
#include "kernels.h"
#include <cstdio>
using namespace linattn;
// width 64: an odd number of workgroups a head only where the even split has one with tiles of two heads, and so saves something
int main() {
  long bad = 0, kept = 0, dealt = 0;
  for (int BH = 1; BH <= 255; ++BH)
    for (int tiles = 1; tiles <= 90; ++tiles) {
      Plan p{};
      p.BH = BH; p.d = 64; p.kind = kPhiHedgehog; p.bf16_math = true;
      Split& s = p.split;
      s.ntile = tiles; s.T = (long long)BH * tiles;
      s.G = (int)(s.T < kSlots ? s.T : kSlots);
      finish_split(s);
      bool two = false;
      for (int g = 0; g < s.G; ++g) two |= split_head(s, split_lo(s, g)) != split_head(s, split_lo(s, g + 1) - 1);
      const int G = s.G;
      deal_state_pass(&p);
      if (s.G == G) { kept += !two && s.T > kSlots; continue; }
      ++dealt;
      bad += s.PS % 2 && !two;
    }
  printf("bad %ld kept %ld dealt %ld\n", bad, kept, dealt);
  return bad != 0 || kept == 0 || dealt == 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_state_pass_keeps_the_even_split_where_no_workgroup_has_two_heads(tmp_path):
    src, exe = tmp_path / "even.cpp", tmp_path / "even"
    src.write_text(EVEN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                    "-I", os.path.join(ROOT, "paper_2510_08318_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


UNITS = r"""
#include "kernels.h"
#include <cstdio>
using namespace linattn;
// states that the workgroups of a call bring into the L2s of eight XCDs
static long long states(const Split& s, int BH, int blocks, int partials) {
  const long long per_head = (blocks + s.blocks - 1) / s.blocks;
  return BH * (per_head < 8 ? per_head : 8) * partials;
}
int main() {
  long bad = 0, held = 0;
  for (int BH : {1, 2, 4, 8, 16, 24, 48, 64, 100, 128, 200, 255})
    for (int blocks : {1, 2, 3, 4, 8, 10, 16, 20, 24, 32, 64, 100})
      for (int partials : {1, 2, 4, 8})
        for (UnitLimits most : {UnitLimits(), UnitLimits{240, 64}, UnitLimits{240, 16}, UnitLimits{240, 0}}) {
          const Split s = make_deal_of_blocks(BH, blocks, 8, {4, 2, 5, 240}, false, partials, most);
          Split t = s, l = s;
          t.blocks = 2 * s.blocks;
          if (s.blocks < 8) bad += states(s, BH, blocks, partials) - states(t, BH, blocks, partials) > (s.blocks == 4 ? most.four : most.two);
          // and no larger than the limits ask for
          l.blocks = s.blocks / 2;
          if (s.blocks > 2 && BH * ((blocks + l.blocks - 1) / l.blocks) <= kCUs) {
            ++held;
            bad += states(l, BH, blocks, partials) - states(s, BH, blocks, partials) <= (l.blocks == 4 ? most.four : most.two);
          }
        }
  printf("bad %ld held %ld\n", bad, held);
  return bad != 0 || held == 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_smaller_units_only_where_the_states_they_read_allow_it(tmp_path):
    src, exe = tmp_path / "units.cpp", tmp_path / "units"
    src.write_text(UNITS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                    "-I", os.path.join(ROOT, "paper_2510_08318_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_every_block_is_dealt_once(tmp_path):
    src, exe = tmp_path / "deal.cpp", tmp_path / "deal"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                    "-I", os.path.join(ROOT, "paper_2510_08318_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
