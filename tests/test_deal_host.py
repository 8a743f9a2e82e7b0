"""The deal of a kernel's units to workgroups (kernels.h: Split, Share, make_deal): the index arithmetic against 128-bit integers, every unit
to one workgroup, at most two heads to a workgroup, and the choice of the deal by its cost."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

PROGRAM = r"""
#include "kernels.h"
#include <cstdio>
#include <cstdlib>
#include <vector>
using namespace linattn;
typedef __int128 wide;
static long bad = 0, even_deals = 0, part_deals = 0;
static void arithmetic(const Split& s) {
  for (int k = 0; k < 40; ++k) {
    const int g = k == 0 ? 0 : k == 1 ? s.G : rand() % (s.G + 1);
    bad += split_lo(s, g) != (long long)((wide)g * s.T / s.G);
    long long x = (long long)(((unsigned long long)rand() << 31 | rand()) % s.T);
    if (k == 2) x = 0;
    if (k == 3) x = s.T - 1;
    if (k % 4 == 0) x = x / s.ntile * s.ntile;
    if (k % 4 == 1) x = x / s.ntile * s.ntile + s.ntile - 1;
    bad += split_head(s, x) != x / s.ntile;
    const int o = split_owner(s, x);
    bad += !(o >= 0 && o < s.G && (wide)o * s.T / s.G <= x && x < (wide)(o + 1) * s.T / s.G);
  }
}
static void cover(const Split& s) {
  std::vector<unsigned char> seen(s.T, 0);
  const dim3 grid = grid_of(s);
  bad += (long long)grid.x * grid.y != s.G;
  for (int gy = 0; gy < (int)grid.y; ++gy)
    for (int gx = 0; gx < (int)grid.x; ++gx) {
      int shares = 0;
      for (Share sh = first_share(s, gx, gy); sh.there; sh = next_share(s, gx, sh), ++shares)
        for (int u = sh.u; u < sh.end; u += sh.step) {
          if (u < 0 || u >= s.ntile || sh.step < 1) { ++bad; break; }
          ++seen[(long long)sh.bh * s.ntile + u];
        }
      bad += shares < 1 || shares > 2;
    }
  for (unsigned char c : seen) bad += c != 1;
}
static int most_units(const Split& s) {
  int most = 0;
  const dim3 grid = grid_of(s);
  for (int gy = 0; gy < (int)grid.y; ++gy)
    for (int gx = 0; gx < (int)grid.x; ++gx) {
      int units = 0;
      for (Share sh = first_share(s, gx, gy); sh.there; sh = next_share(s, gx, sh)) units += (sh.end - sh.u + sh.step - 1) / sh.step;
      most = units > most ? units : most;
    }
  return most;
}
int main() {
  const int heads[] = {1, 2, 3, 5, 7, 12, 13, 24, 30, 40, 87, 128, 129, 255, 256, 257, 1000, 65535};
  const int units[] = {1, 2, 3, 4, 5, 7, 8, 9, 16, 21, 22, 64, 65, 128, 255, 256, 257, 296, 1000, 9451};
  for (int BH : heads)
    for (int per : units)
      for (int c : {0, 3, 8}) {
        const Split s = make_deal(BH, per, {c});
        arithmetic(s);
        even_deals += !s.share;
        if (s.T < 400000) cover(s);
        if (s.T < 400000 && BH < kCUs) {
          const int share = kCUs / BH < per ? kCUs / BH : per, by_head = (per + share - 1) / share;
          bad += s.G > kCUs || most_units(s) > by_head;
          bad += !s.share && 8 * most_units(s) + c >= 8 * by_head;        // the second prologue has to pay
        }
      }
  // rounds for a part of the compute units that cost less: still every unit once, and never more units to a workgroup than head by head
  for (int BH : heads)
    for (int per : units) {
      const Split s = make_deal(BH, per, {4, 2, 5, 240});
      arithmetic(s);
      if (s.T >= 400000) continue;
      cover(s);
      if (BH >= kCUs) continue;
      const int share = kCUs / BH < per ? kCUs / BH : per, by_head = (per + share - 1) / share;
      bad += s.G > kCUs || most_units(s) > by_head;
      part_deals += s.share != make_deal(BH, per, {4}).share;
    }
  // kernels without the loop over a workgroup's heads: a head to a workgroup at every length up to the largest n (2^30 tokens), where the even deal would
  // save any number of rounds
  for (int BH : heads)
    for (int per : {1, 2, 3, 255, 256, 1000, 1 << 17, 1 << 18, 1 << 20, 1 << 22}) {
      const Split s = make_deal(BH, per, {3}, false);
      bad += s.share < 1 || s.G != BH * s.share;
      if (s.share < 1) continue;
      arithmetic(s);
      if (s.T < 400000) cover(s);
    }
  for (int k = 0; k < 3000; ++k) {                       // large counts: only the arithmetic
    Split s{};
    s.ntile = 1 + rand() % 33554432;
    const int BH = 1 + rand() % (k % 2 ? 256 : 65535);
    s.T = (long long)BH * s.ntile;
    s.G = BH > 256 ? BH : s.T < 256 ? (int)s.T : 256;
    finish_split(s);
    arithmetic(s);
  }
  printf("bad %ld even %ld part %ld\n", bad, even_deals, part_deals);
  return bad != 0 || even_deals == 0 || part_deals == 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_every_unit_is_dealt_once(tmp_path):
    src, exe = tmp_path / "deal.cpp", tmp_path / "deal"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                    "-I", os.path.join(ROOT, "paper_2510_08318_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
