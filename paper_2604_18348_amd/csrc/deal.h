// Sparse launches whose tiles are dealt to the XCDs by work: which they are, and the sizes of their lists (attn.hip; also compiled for the CPU).
#pragma once
#include <cstdint>

namespace adac {

static constexpr int F32_MAX_SPLITS = 4; // most workgroups the fp32 kernel splits a key list over
__host__ __device__ constexpr int f32_resident(int d) { return 32 * (d == 64 ? 3 : 2); }   // of its workgroups on the 32 CUs of an XCD
constexpr int PICK_HEADS = 256;          // heads up to which the tiles of a launch are one list (pick_tile in attn.hip)
// Most pieces a key list of the fp32 kernel may go in (see pick_tile).  From some 1 024 tiles on there are two rounds of whole
// ones (d=128), and the partial results of every row and the launch that combines them cost what the last round leaves idle
// (150 heads of 200 rows: 58 us whole, 66 in pieces).
inline int f32_splits(int H, int N, int Cq) { return H <= PICK_HEADS && (long long)H * (N / 32 + Cq / 2 + 1) < 1024 ? F32_MAX_SPLITS : 1; }

constexpr int PLAN_BESIDE = 256;       // query clusters up to which the LDS of the plan (9 KB, and 11 KB at 256) leaves a CU its eight workgroups of plan_sparse
constexpr int DEAL_ENTRIES = 64;                     // segments at most
// A head's record: the longest list (key tiles) of every segment, the first tile of every part of the segments and the end
__host__ __device__ constexpr int deal_rec(int segs) { return segs + 8 * segs + 1; }
constexpr int DEAL_PARTS = 10 * DEAL_ENTRIES;        // of all heads: H * segs <= DEAL_ENTRIES
constexpr int DEAL_HEAD = 4;                         // an XCD's list: their number (and padding), the entries
__host__ __device__ constexpr int deal_cap(int tiles) { return tiles * 9 / 64 + 2; }       // most tiles of a part, of `tiles` in eight parts
// First tiles of a segment's eight parts and its end, as near to those of equal work as no part has more than that.
__host__ __device__ inline void deal_parts(int (&at)[9]) {
  const int cap = deal_cap(at[8] - at[0]);
  for (int x = 1; x < 8; ++x) {
    const int least = at[8] - (8 - x) * cap, most = at[x - 1] + cap < at[8] ? at[x - 1] + cap : at[8];
    int b = at[x] > at[x - 1] ? at[x] : at[x - 1];
    if (b < least) b = least;
    at[x] = b < most ? b : most;
  }
}
// Most tiles of an XCD, of at most `most` a head: the grid of a launch is what its lists can hold, as every workgroup without an entry takes a
// place and a trip to memory.
inline int deal_list(int H, int segs, int most) { return H * (most * 9 / 64 + 2 * segs); }
// Most entries of an XCD, fp32, where lists may go in pieces: all of them while the tiles are one round, those past the last whole round else.
inline int deal_entries_f32(int d, int H, int N, int Cq, int segs, int most) {
  const int tiles = deal_list(H, segs, most), round = f32_resident(d);
  if (f32_splits(H, N, Cq) == 1) return tiles;
  return tiles <= round ? F32_MAX_SPLITS * tiles : tiles + (F32_MAX_SPLITS - 1) * round;
}

inline int deal_segs(int H, int tiles) { const int n = DEAL_ENTRIES / H < 8 ? DEAL_ENTRIES / H : 8, m = n < tiles / 16 ? n : tiles / 16; return m > 1 ? m : 1; }
// Segments a head where the tiles of a sparse launch are dealt by work; 0 where by their number.  Dealt by number, an XCD has what its heads
// happen to have.  Calls, by number -> by work: 16 x 14 119, d=128, some heads without structure 888 -> 844 us, 30 x 21 600, d=64, top-p 862 -> 772,
// 16 x 22 680, d=64, 93 clusters, a later step 1 703 -> 1 339, 8 x 6 000, d=128 233 -> 222, 4 x 13 200, d=128 403 -> 390, 16 x 6 000, d=64 232 -> 214,
// 5 x 9 247, d=128, entry points one by one 528 -> 505; heads of equal lists, 30 x 17 776, 1 397 and 1 397; of 67 top-k calls 0.977, none more than 1.013.
// The plan takes 4-6 us more (its last head waits for three trips to memory): a tile a CU (n < 256) or short lists (under 75 key tiles a place) give it
// back here and there (ten such calls 0.96 ... 1.04: 3 x 5 000, d=128 215 -> 208, 23 x 1 680, d=128 227 -> 230, 6 x 4 000, d=128, top-p 219 -> 227), and from
// sixteen rounds on the ends of the lists are less than that.
constexpr double DEAL_MIN = 75;      // key tiles (of a list of all keys) a place
inline int deal_segs_bf16(int BM, int resident /* workgroups of the chip */, int H, int N, int Cq) {
  if (Cq < 2 || Cq > PLAN_BESIDE || H > DEAL_ENTRIES) return 0;
  const int tiles = N / BM + Cq / 2 + 1, T = (N + 63) / 64;
  const double n = (double)H * tiles, r = resident;
  if (n < 256 || n >= 16 * r || n * T < DEAL_MIN * r || 9.0 * H * (N / BM + Cq + 1) * (T + 64.0) >= 2147483648.0) return 0;
  return deal_segs(H, tiles);
}
// fp32: key tiles (of a list of all keys) a CU, by width.  Lists of uneven length are what is to be gained: calls of 4 x 8 208, d=64 384 ->
// 368 us, of 4 x 8 208, d=128 638 -> 600, top-p 761 -> 688, 3 x 9 710, d=128 684 -> 662, 4 x 11 000, d=128, top-p 921 -> 795.
// While the tiles are one round only top-p lists are so uneven that it pays for the plan (7 us): 2 x 6 437, d=128 405 -> 297, 2 x 8 000, d=64
// 299 -> 269, 1 x 12 000, d=128 479 -> 454; top-k 2 x 6 437 306 -> 315, a later step 233 -> 243, 2 x 8 000, d=64 284 -> 288, 2 x 10 944, d=64, a later step
// 279 -> 286, 1 x 9 500, d=128 392 -> 404 (of 59 such calls 1.009, 0.95 ... 1.06; 1 x 12 000, d=128, a later step 342 -> 331).  At d=128 the tiles
// dealt by number have the same pieces past the whole round between one and 1.9 rounds: 18 calls 1.00 (3 x 7 920, a later step 365 -> 359, 3 x 5 007, a later step 235 -> 237,
// 2 x 8 160 453 -> 462, top-p 531 -> 554); at d=64 1.1 rounds are already worth it (3 x 8 000, top-p 419 -> 361, top-k 334 -> 333, a later step 249 -> 248).
constexpr double F32_DEAL_MIN_64 = 200, F32_DEAL_MIN_128 = 165;
inline int deal_segs_f32(int d, int H, int N, int Cq, bool top_p) {
  if (Cq < 2 || Cq > PLAN_BESIDE || H > DEAL_ENTRIES) return 0;
  const int tiles = N / 32 + Cq / 2 + 1, T = (N + 63) / 64;
  if (tiles > 65536 || (double)H * tiles * T < 256 * (d == 64 ? F32_DEAL_MIN_64 : F32_DEAL_MIN_128) || 4.0 * H * (N / 32 + Cq + 1) * (T + 64.0) >= 2147483648.0) return 0;
  const double rounds = (double)H * tiles / (8 * f32_resident(d));
  if ((!top_p && rounds <= 1) || (d == 128 && rounds > 1 && rounds < 1.9)) return 0;
  return deal_segs(H, tiles);
}

}  // namespace adac
