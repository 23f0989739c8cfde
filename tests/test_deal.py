"""The lists of tiles dealt to the XCDs by work: their sizes against every deal they may have to hold, compiled for the CPU."""
import os
import subprocess

import pytest

from paper_2604_18348_amd import binding as B
from tests import test_gpu_attention as attention

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
    const int segs = f32 ? deal_segs_f32(d, H, N, Cq, upto(1)) : deal_segs_bf16(BM, 256 * (BM == 128 ? 2 : 1) * (d == 64 ? 2 : 1), H, N, Cq);
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
  const int big = 8 * deal_entries_f32(64, 3, 10876, 65, deal_segs_f32(64, 3, 10876, 65, false), 10876 / 32 + 66);
  if (big > 1800) { std::printf("3 x 10 876: %d workgroups for some 1 100 tiles\n", big); return 1; }
  return worst < 2.2 && dealt > 2000 ? 0 : 1;
}
"""


RULES = r"""
#include <cstdio>
#define __host__
#define __device__
#include "deal.h"
using namespace adac;
int main() {
  int f32, H, N, d, Cq;
  while (std::scanf("%d %d %d %d %d", &f32, &H, &N, &d, &Cq) == 5) {
    const int BM = N / Cq < 768 ? 128 : 256;
    if (f32) std::printf("%d %d\n", deal_segs_f32(d, H, N, Cq, false), deal_segs_f32(d, H, N, Cq, true));
    else { const int s = deal_segs_bf16(BM, 256 * (BM == 128 ? 2 : 1) * (d == 64 ? 2 : 1), H, N, Cq); std::printf("%d %d\n", s, s); }
  }
}
"""


def compiled(tmp_path, program):
    src, exe = tmp_path / "deal.cpp", tmp_path / "deal"
    src.write_text(program)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2604_18348_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, timeout=120)
    return str(exe)


def test_lists_hold_every_deal_and_little_more(tmp_path):
    out = subprocess.run([compiled(tmp_path, PROGRAM)], stdout=subprocess.PIPE, text=True, timeout=100)
    assert out.returncode == 0, out.stdout
    print(out.stdout)


def shapes_of(test):
    return [tuple(s) for m in test.pytestmark if m.name == "parametrize" for s in m.args[1]]


def test_which_launches_are_dealt(tmp_path):
    """The shapes that the GPU tests of dealt tiles take are dealt; fp32 launches of one round of tiles are for top-p alone."""
    bf16 = [(0, *s) for s in shapes_of(attention.test_tiles_dealt_by_work)]
    f32 = [(1, *s) for s in shapes_of(attention.test_fp32_tiles_dealt_by_work)]
    fused = [s for s in attention.FUSED_DEALT] + [(*s, "topp") for s in attention.DEAD_DEALT]
    bf16 += [s[:5] for s in fused if not s[0]]
    f32 += [s[:5] for s in fused if s[0]]
    whole = [s[:5] for s in fused if s[5] == "topk"]
    one_round = [(1, 2, 6437, 128, 65), (1, 2, 6522, 128, 65), (1, 2, 8000, 64, 65), (1, 2, 10944, 64, 65), (1, 1, 9500, 128, 65)]
    by_number = [(1, 3, 5007, 128, 65), (1, 2, 8160, 128, 65), (1, 4, 8208, 128, 1), (0, 65, 9000, 64, 65), (0, 5, 9247, 128, 257)]
    asked = bf16 + f32 + one_round + by_number
    out = subprocess.run([compiled(tmp_path, RULES)], input="\n".join(" ".join(map(str, s)) for s in asked), stdout=subprocess.PIPE, text=True,
                         timeout=60, check=True)
    for s, line in zip(asked, out.stdout.splitlines()):
        topk, topp = map(int, line.split())
        assert (topp > 0) == (s not in by_number) and (topk == 0 or s not in one_round) and (topk > 0 or s not in bf16 + whole), (s, line)


@pytest.mark.parametrize("H,N,d", [(2, 6437, 128), (3, 10876, 64), (2, 8000, 64)])
def test_one_workspace_for_either_selection(H, N, d):
    size = [B.adacluster_workspace_bytes(B.Params(H=H, N=N, d=d, dtype=B.F32, q_clusters=65, k_m0=32, k_max_clusters=256, select_mode=m))
            for m in (B.SELECT_TOPK, B.SELECT_TOPP)]
    assert size[0] == size[1]
