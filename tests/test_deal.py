"""The lists of tiles dealt to the XCDs by work: their sizes against every deal they may have to hold, compiled for the CPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>
#define __host__
#define __device__
#include "deal.h"
using namespace adac;
static std::mt19937_64 rng(1);
static int upto(int n) { return (int)(rng() % (unsigned)(n + 1)); }
static long long checked;

// One deal of a launch whose heads have at most `most` tiles: the parts as the plan forms them, of arbitrary equal-work boundaries, and an
// XCD's entries for every way its lists may go in pieces.
static void deal(bool f32, int d, int H, int N, int Cq, int segs, int most, int entries) {
  std::vector<int> of_xcd(8, 0);
  for (int h = 0; h < H; ++h) {
    const int nt = upto(3) ? most - upto(most / 8) : upto(most);
    std::vector<int> cuts(segs + 1, nt);
    cuts[0] = 0;
    for (int s = 1; s < segs; ++s) cuts[s] = upto(nt);
    std::sort(cuts.begin(), cuts.end());
    for (int s = 0; s < segs; ++s) {
      int at[9], first = cuts[s], end = cuts[s + 1];
      const int kind = upto(3);
      at[0] = first; at[8] = end;
      for (int x = 1; x < 8; ++x) at[x] = kind == 0 ? first : kind == 1 ? end : first + upto(end - first);
      std::sort(at, at + 9);
      deal_parts(at);
      if (at[0] != first || at[8] != end) { std::printf("parts lose tiles\n"); std::exit(1); }
      for (int x = 0; x < 8; ++x) {
        if (at[x + 1] < at[x] || at[x + 1] - at[x] > deal_cap(end - first)) { std::printf("a part of %d of %d tiles\n", at[x + 1] - at[x], end - first); std::exit(1); }
        of_xcd[x] += kind == 3 ? at[x + 1] - at[x] : deal_cap(end - first) < end - first ? deal_cap(end - first) : end - first;      // (the rotation may give an XCD the largest part of each)
      }
    }
  }
  const bool cut = f32 && f32_splits(H, N, Cq) > 1;
  const int round = f32_resident(d);
  for (int x = 0; x < 8; ++x) {
    const int n = of_xcd[x];
    const int need = !cut ? n : n <= round ? n * F32_MAX_SPLITS : n - n % round + n % round * F32_MAX_SPLITS;
    if (need > entries) { std::printf("f32 %d d %d H %d N %d Cq %d: %d entries for %d\n", f32, d, H, N, Cq, entries, need); std::exit(1); }
    ++checked;
  }
}

int main() {
  double worst = 0;
  int dealt = 0;
  for (int i = 0; i < 40000; ++i) {
    const bool f32 = i & 1;
    const int d = upto(1) ? 64 : 128, H = 1 + upto(upto(1) ? 8 : 63), Cq = 2 + upto(upto(3) ? 98 : 254), N = std::max(Cq, (int)(600 * std::pow(300.0, upto(1000) / 1000.0)));
    const int BM = f32 ? 32 : N / Cq < 768 ? 128 : 256;
    const int segs = f32 ? deal_segs_f32(d, H, N, Cq) : deal_segs_bf16(BM, 256 * (BM == 128 ? 2 : 1) * (d == 64 ? 2 : 1), H, N, Cq);
    if (!segs) continue;
    ++dealt;
    if (H * segs > DEAL_ENTRIES || segs > 8 || H * deal_rec(segs) > DEAL_PARTS) { std::printf("records of %d heads, %d segments\n", H, segs); return 1; }
    const int most = N / BM + Cq + 1 + (f32 ? 0 : 128);
    const int entries = f32 ? deal_entries_f32(d, H, N, Cq, segs, most) : deal_list(H, segs, most);
    // the workgroups of the launch against the tiles, and pieces of what is past a whole round (or of all, while they are less than one), that there can be
    const int tiles = H * most, all = 8 * f32_resident(d);
    const double there = f32 && f32_splits(H, N, Cq) > 1 ? (tiles <= all ? F32_MAX_SPLITS * tiles : tiles + (F32_MAX_SPLITS - 1) * all) : tiles;
    worst = std::max(worst, 8.0 * entries / there);
    for (int k = 0; k < 3; ++k) deal(f32, d, H, N, Cq, segs, most, entries);
  }
  std::printf("%d launches, %lld lists, at most %.2f workgroups a tile\n", dealt, checked, worst);
  const int big = 8 * deal_entries_f32(64, 3, 10876, 65, deal_segs_f32(64, 3, 10876, 65), 10876 / 32 + 66);
  if (big > 1800) { std::printf("3 x 10 876: %d workgroups for some 1 100 tiles\n", big); return 1; }
  return worst < 2.2 && dealt > 2000 ? 0 : 1;
}
"""


def test_lists_hold_every_deal_and_little_more(tmp_path):
    src, exe = tmp_path / "deal.cpp", tmp_path / "deal"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2604_18348_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, timeout=120)
    out = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True, timeout=100)
    assert out.returncode == 0, out.stdout
    print(out.stdout)
