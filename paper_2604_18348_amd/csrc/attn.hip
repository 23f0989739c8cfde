// Attention over the selected key clusters (Alg. 3 lines 9-10) and the dense branch.
//
// The label sort puts the keys in cluster order (a permutation, no copy: the planning step writes, per query
// cluster, where every selected key row sits in K and V as they are, and the kernels load their tiles through
// that table).  For
// every query cluster the selected key clusters form a short list of row ranges in that order; a
// query tile walks the concatenation of its ranges in full 64-key tiles, so cluster raggedness
// costs nothing but one masked tail tile.  The flash-style kernel keeps the S^T = K Q^T
// orientation: in the 32x32 MFMA accumulator a lane then owns one query and 16 keys, soft-max
// statistics are per-lane scalars, and the exponentiated block feeds the P V product as the B
// operand straight from registers.  K and V tiles both sit row-major in LDS; the A operand of that
// product (a column of V over 8 keys) is gathered by LDS transpose reads.
#include "common.h"
#include "launch.h"
#include "deal.h"

#include <type_traits>

namespace adac {

static constexpr int TILE_REC = 8;       // ints per query-tile record (32 bytes)
static constexpr int MIN_CHUNK = 16;     // key tiles of a chunk at least: lists of up to twice as many stay whole
static constexpr int SPLIT_SLOTS = 128;  // partial slots per head for the chunks of cut key lists
static constexpr int F32_WAVES = 4;      // waves of a workgroup of the fp32 kernel
static constexpr float PART_DONE = -1.f; // in place of the sum of a row's first partial result: the row is written
static constexpr int KROW_PAD = 8 * 64;  // entries of the row-offset table a key list is padded by: the kernel reads up to 7 tiles ahead

// ------------------------------------------------------------------------------------------
// plan: per query cluster the merged key ranges; per head the list of query tiles
// ------------------------------------------------------------------------------------------
// rng_start [H][Cq][maxr]   first key row (in cluster order) of range r
// rng_pre   [H][Cq][maxr+1] keys before range r in the concatenation (last = total)
// rng_cnt   [H][Cq]
// tiles     [H][maxtiles] x {cluster, first sorted query position, rows, first key tile, end key
//           tile, partial slot or -1, keys of the cluster's whole list, not 0: the second 32 rows of 64 (fp32)}; ntiles [H]
__device__ __forceinline__ int wave_prefix(int v, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) { const int u = __shfl_up(v, o); if (lane >= o) v += u; }
  return v;
}

// Query tiles of a head, cluster by cluster.  A query cluster whose key list is much longer than
// the head's average (top-p selections can be that skewed) would make its few workgroups the whole
// critical path of the launch, so such a list is cut into chunks of key tiles: each chunk is a
// workgroup of its own that leaves unnormalised (O, m, l) in a partial slot, and attn_merge
// combines the slots of a query tile.  merge [H][slots] x {first query position, rows, first slot,
// chunks}; a head has `slots` partial slots, and lists stay whole once they are used up.
__host__ __device__ constexpr int plan_ints(int Cq, bool deal) { return (deal ? 11 : 9) * Cq + 1; }      // of LDS
// Pieces for `rest` tiles of an XCD, for every number of them: two bits each (pieces - 1), 32 a word.  By the host, as the
// kernel's registers and first microseconds are dear (3 x 5 007 rows, d=128, a call 288 us, 290 with the rule in the kernel).
struct Pieces { uint64_t of[3]; };
__device__ __forceinline__ int pieces_of(const Pieces& p, int rest) {
  const uint64_t w = rest < 32 ? p.of[0] : rest < 64 ? p.of[1] : p.of[2];
  return 1 + (int)(w >> (2 * (rest & 31)) & 3);
}

// Tiles dealt to the XCDs by work (attn_deal_segs says when).  Workgroups go to the 8 XCDs in turn, and one is done when the last is.
// The query clusters of a head are ordered by the length of their key lists, the longest first, and their tiles cut into `segs`
// segments of equal work, each in eight parts of equal work, one for every XCD (the tiles of a cluster stay side by side); segment e's
// parts are dealt from XCD e % 8 on, so that what rounding leaves evens out.  The last head to be planned writes every XCD's list: its
// parts of all segments, the longest lists first, whatever head they are of, so that what ends last is short.  A bf16 tile is run as
// its record says, so that a head's bits do not depend on the other heads (in launches of less than two rounds the tiles past the last
// whole one went in pieces: calls of 8 x 6 000, d=128 222 -> 241 us, 7 x 8 000, d=128 220 -> 237, and 5 x 9 247 505 -> 481).
// Fp32 lists go in pieces as in pick_tile, or, where all are one round, each in pieces of about a sixth of a CU's work (2 x 6 437
// top-p, d=128, by number 166 us, so 62; in launches of more rounds pieces of every list cost more than they even out: 3 x 5 007 177 -> 203).
struct DealtTile { int h, tile, z, sp; };            // head, tile, piece and (fp32) of how many
__device__ __forceinline__ int dealt(int h, int tile, int z, int sp = 1) { return h << 23 | tile << 6 | z << 3 | (sp - 1); }
__device__ __forceinline__ DealtTile dealt_tile(uint32_t e) { return {(int)(e >> 23), (int)(e >> 6 & 0x1FFFF), (int)(e >> 3 & 7), (int)(e & 7) + 1}; }      // (tile: 17 bits)
struct Deal { int32_t* parts /* [H][deal_rec(segs)] */; int32_t* lists /* [8][DEAL_HEAD + cap] */; int32_t* planned /* heads; 0 before the launch */; int cap, segs, H; int f32_round /* fp32: workgroups of an XCD at a time, where lists may be cut */; Pieces pieces; };

// By the workgroup of the last head to be planned.
__device__ __forceinline__ void deal_lists(const Deal& dl) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int H = dl.H, segs = dl.segs, rec = deal_rec(segs), E = H * segs;
  constexpr int ROUNDS = (DEAL_PARTS + 255) / 256;
  __shared__ int32_t s_part[ROUNDS * 256], s_rank[DEAL_ENTRIES], s_by_rank[DEAL_ENTRIES];
  {
    int32_t v[ROUNDS];                               // (asked for together)
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) v[r] = __hip_atomic_load(dl.parts + min(tid + r * 256, H * rec - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) s_part[tid + r * 256] = v[r];
    if (tid < DEAL_ENTRIES) s_rank[tid] = 0;
  }
  lds_barrier();
  {                                                  // segments ahead of every segment, a quarter of them by every wave
    const int key = lane < E ? s_part[lane / segs * rec + lane % segs] << 6 | (63 - lane) : 0;       // (no two alike)
    int rank = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) rank += __builtin_amdgcn_readlane(key, wave * 16 + j) > key;
    atomicAdd(&s_rank[lane], rank);
  }
  lds_barrier();
  if (tid < E) s_by_rank[s_rank[tid]] = tid;
  lds_barrier();
  const int e = lane < E ? s_by_rank[lane] : 0, h = e / segs;      // a lane a segment, in order
  const int32_t* const p = s_part + h * rec + segs + (e - h * segs) * 8;
  for (int xcd = wave; xcd < 8; xcd += 4) {          // a wave an XCD
    const int y = (xcd + e) & 7, first = p[y], n = lane < E ? p[y + 1] - first : 0;
    const int tiles = __builtin_amdgcn_readlane(wave_prefix(n, lane), 63);
    int cut = 1;                                     // pieces of this segment's lists
    if (dl.f32_round && tiles <= dl.f32_round) {     // fp32, one round of workgroups: pieces of about a sixth of a CU's work
      const int T = lane < E ? p[-segs - 7 * (e - h * segs)] : 0;      // (the segment's longest list: the record starts with those)
      const int chunk = max(4, __builtin_amdgcn_readlane(wave_prefix(n * T, lane), 63) / (32 * 6));
      cut = min(F32_MAX_SPLITS, max(1, (T + chunk - 1) / chunk));
    }
    const int mine = n * cut, incl = wave_prefix(mine, lane), total = __builtin_amdgcn_readlane(incl, 63);
    int rest = 0, sp = 1;
    if (dl.f32_round) {                              // more: those past the last whole round in pieces, as in pick_tile
      if (tiles > dl.f32_round) rest = (uint32_t)total % (uint32_t)dl.f32_round;
      if (rest) sp = pieces_of(dl.pieces, rest);
    }
    const int whole = total - rest;
    int32_t* const list = dl.lists + (size_t)xcd * (DEAL_HEAD + dl.cap);
    if (lane == 0) list[0] = whole + rest * sp;
    if (cut > 1) {
      for (int i = 0; i < n; ++i)
        for (int z = 0; z < cut; ++z) list[DEAL_HEAD + incl - mine + z * n + i] = dealt(h, first + i, z, cut);
    } else {
      for (int i = 0; i < n; ++i) {
        const int s = incl - n + i;
        if (s < whole) { list[DEAL_HEAD + s] = dealt(h, first + i, 0); continue; }
        for (int z = 0; z < sp; ++z) list[DEAL_HEAD + s + z * rest] = dealt(h, first + i, z, sp);
      }
    }
  }
}

template <bool KNOWN, bool DEAL>
__device__ __forceinline__ void tiles_of_head(int32_t* sm, int h, int Cq, int maxr, int maxtiles, int BM, int slots, int allow_split, const Deal& dl,
                                              const int32_t* __restrict__ q_offs, int q_offs_stride, const int32_t* __restrict__ lengths,
                                              const int32_t* __restrict__ rng_pre, const int32_t* __restrict__ rng_cnt,
                                              int32_t* __restrict__ tiles, int32_t* __restrict__ ntiles,
                                              int32_t* __restrict__ merge, int32_t* __restrict__ nmerge) {
  const int tid = threadIdx.x, C = Cq;
  const int32_t* qo = q_offs + (size_t)h * q_offs_stride;
  int32_t* tl = tiles + (size_t)h * maxtiles * TILE_REC;
  int32_t* ml = merge + (size_t)h * slots * 4;
  int32_t *const s_T = sm, *const s_nq = sm + C, *const s_pieces = sm + 2 * C, *const s_tile0 = sm + 3 * C, *const s_slot0 = sm + 4 * C,
          *const s_merge0 = sm + 5 * C, *const s_tot = sm + 6 * C, *const s_list = sm + 7 * C;
  int32_t* const s_q0 = sm + 8 * C;                                                 // [C + 1] first rows
  int32_t *const s_order = sm + 9 * C + 1, *const s_work = sm + 10 * C + 1;         // (dealt: the clusters in their order, the work before each)
  const auto at_place = [&](int i) __attribute__((always_inline)) { if constexpr (DEAL) return s_order[i]; else return i; };
  for (int c = tid; c < C; c += 256) {
    const int q0 = qo[c], q1 = qo[c + 1];
    s_nq[c] = (q1 - q0 + BM - 1) / BM;
    s_q0[c] = q0;
    if (c == C - 1) s_q0[C] = q1;
    int tot;
    if constexpr (KNOWN) tot = lengths[(size_t)h * Cq + c];
    else tot = rng_pre[((size_t)h * Cq + c) * (maxr + 1) + rng_cnt[(size_t)h * Cq + c]];
    s_T[c] = (tot + 63) / 64;
    s_tot[c] = tot;
  }
  __syncthreads();
  // A thread looks after the clusters tid * per .., so that prefix sums over the threads are in cluster order.  Only the
  // lists that are cut are dealt with one after the other (all of them by one thread: 15 us at 65 clusters, now 6).
  const int per = (C + 255) / 256, c0 = min(C, tid * per), c1 = min(C, c0 + per), lane = tid & 63, wave = tid >> 6;
  __shared__ long long w_work[4];
  __shared__ int32_t w_a[4], w_b[4];
  __shared__ int32_t s_cut, s_ntiles, s_last;
  {
    // key tiles per chunk of a list that is cut: twice the average list of the head, at least 16
    long long work = 0; int qtiles = 0;
    for (int c = c0; c < c1; ++c) { work += (long long)s_nq[c] * s_T[c]; qtiles += s_nq[c]; }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) { work += __shfl_xor(work, o); qtiles += __shfl_xor(qtiles, o); }
    if (lane == 0) { w_work[wave] = work; w_a[wave] = qtiles; }
  }
  __syncthreads();
  const long long work = w_work[0] + w_work[1] + w_work[2] + w_work[3];
  const int qtiles = w_a[0] + w_a[1] + w_a[2] + w_a[3];
  const int chunk = max(MIN_CHUNK, 2 * (qtiles > 0 ? (int)((work + qtiles - 1) / qtiles) : 0));
  // which lists are cut: the long ones are listed in cluster order, and one thread deals the slots out while they last
  int cuts = 0;
  for (int c = c0; c < c1; ++c) { s_pieces[c] = 1; cuts += allow_split && s_T[c] > 2 * chunk; }
  const int cin = wave_prefix(cuts, lane);
  if (lane == 63) w_b[wave] = cin;
  __syncthreads();
  {
    int at = cin - cuts;
    for (int w = 0; w < wave; ++w) at += w_b[w];
    for (int c = c0; c < c1; ++c) if (allow_split && s_T[c] > 2 * chunk) s_list[at++] = c;
    if (tid == 255) s_cut = at;
  }
  __syncthreads();
  if (tid == 0) {
    int used = 0, nm = 0;
    for (int i = 0; i < s_cut; ++i) {
      const int c = s_list[i], T = s_T[c];
      int pieces = min(16, (T + chunk - 1) / chunk);
      if (used + pieces * s_nq[c] > slots) pieces = max(1, (slots - used) / max(s_nq[c], 1));   // fewer, longer chunks
      if (pieces > 1) {
        const int per_piece = (T + pieces - 1) / pieces;
        pieces = max(1, (T + per_piece - 1) / max(per_piece, 1));          // no empty chunk
      }
      s_pieces[c] = pieces; s_slot0[c] = used; s_merge0[c] = nm;
      if (pieces > 1) { used += s_nq[c] * pieces; nm += s_nq[c]; }
    }
    nmerge[h] = nm;
  }
  __syncthreads();
  // What a tile takes: its key tiles and about four steps for start and end, and of a step a share that does not depend on how many
  // of its waves have rows.
  const auto step_of = [&](int rows) __attribute__((always_inline)) { return (rows + 31) / 32 + 1; };
  const auto work_of = [&](int c, int& group) __attribute__((always_inline)) {      // of a cluster, and of BM of its rows
    const int nq = s_nq[c], len = s_T[c] + 4 * s_pieces[c], last = s_q0[c + 1] - s_q0[c] - (nq - 1) * BM;
    group = len * step_of(BM);
    return nq > 0 ? (nq - 1) * group + len * step_of(last) : 0;
  };
  if constexpr (DEAL) {
    __shared__ __attribute__((aligned(16))) int32_t s_key[PLAN_BESIDE];
    const int mine = tid < C ? s_T[tid] << 8 | (255 - tid) : -1;      // (no two alike)
    s_key[tid] = mine;
    lds_barrier();
    int place = 0;
#pragma unroll 4
    for (int o = 0; o < C; o += 4) {
      const int4 k = *reinterpret_cast<const int4*>(&s_key[o]);
      place += (k.x > mine) + (k.y > mine) + (k.z > mine) + (k.w > mine);
    }
    if (tid < C) s_order[place] = tid;
    lds_barrier();
  }
  {                                              // where every cluster's records start
    int mine = 0, work = 0, g;
    for (int i = c0; i < c1; ++i) {
      const int c = at_place(i);
      mine += s_nq[c] * s_pieces[c];
      if constexpr (DEAL) work += work_of(c, g);
    }
    const int incl = wave_prefix(mine, lane), wincl = DEAL ? wave_prefix(work, lane) : 0;
    if (lane == 63) { w_a[wave] = incl; w_b[wave] = wincl; }
    __syncthreads();
    int nt = incl - mine, wt = wincl - work;
    for (int w = 0; w < wave; ++w) { nt += w_a[w]; wt += w_b[w]; }
    for (int i = c0; i < c1; ++i) {
      const int c = at_place(i);
      s_tile0[i] = nt; nt += s_nq[c] * s_pieces[c];
      if constexpr (DEAL) { s_work[i] = wt; wt += work_of(c, g); }
    }
    if (tid == 255) { ntiles[h] = nt; s_ntiles = nt; s_cut = wt; }
  }
  __syncthreads();
  if constexpr (DEAL) {
    __shared__ int32_t s_bound[8 * 8 + 1], s_longest[8];      // (of at most eight segments)
    const int total = s_cut, nt = s_ntiles, segs = dl.segs, an = total / (8 * segs), over = total - an * 8 * segs;
    for (int k = tid; k <= 8 * segs; k += 256) {
      const int want = an * k + over * k / (8 * segs);
      int lo = 0, hi = C - 1;                    // the last cluster whose work starts at or before it
      while (lo < hi) { const int mid = (lo + hi + 1) >> 1; if (s_work[mid] <= want) lo = mid; else hi = mid - 1; }
      const int c = s_order[lo], nq = s_nq[c], pieces = s_pieces[c];
      int group, at = 0;
      (void)work_of(c, group);
      if (nq > 0) at = min((int)((float)(want - s_work[lo]) / (float)group * (float)pieces + 0.5f), nq * pieces);      // (to the nearest tile)
      s_bound[k] = k == 0 ? 0 : k == 8 * segs ? nt : s_tile0[lo] + at;
      if (k % 8 == 0 && k < 8 * segs) s_longest[k / 8] = s_T[c];
    }
    lds_barrier();
    if (tid < 64) {
      int32_t* d = dl.parts + (size_t)h * deal_rec(segs);
      const auto put = [&](int i, int v) __attribute__((always_inline)) { __hip_atomic_store(d + i, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
      if (tid < segs) {
        int at[9];
#pragma unroll
        for (int x = 0; x <= 8; ++x) at[x] = s_bound[8 * tid + x];
        deal_parts(at);
        put(tid, s_longest[tid]);
#pragma unroll
        for (int x = 0; x < 8; ++x) put(segs + 8 * tid + x, at[x]);
      }
      if (tid == 63) put(9 * segs, nt);
      // The stores go through to where every XCD sees them, and have arrived when they are counted: the head reports only then.  (A
      // release fence instead writes back all that the lists' workgroups have left in the L2, 8-12 us.)
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    lds_barrier();
    if (tid == 0) s_last = __hip_atomic_fetch_add(dl.planned, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == dl.H - 1;
  }
  // The records, one a thread: the last cluster whose records start at or before it (an empty one shares its start with
  // the next).  One thread per cluster wrote 625 records one after the other where 20 000 rows are a single cluster.
  for (int t = tid; t < s_ntiles; t += 256) {
    int lo = 0, hi = C - 1;
    while (lo < hi) { const int mid = (lo + hi + 1) >> 1; if (s_tile0[mid] <= t) lo = mid; else hi = mid - 1; }
    const int c = at_place(lo), i = t - s_tile0[lo], T = s_T[c], pieces = s_pieces[c], per_piece = (T + pieces - 1) / pieces;
    const int group = i / pieces, k = i - group * pieces;                    // rows group * BM .. of the cluster, chunk k
    const int r0 = s_q0[c] + group * BM, rows = min(BM, s_q0[c + 1] - r0);
    int32_t* t6 = tl + (size_t)t * TILE_REC;
    t6[0] = c; t6[1] = r0; t6[2] = rows;
    t6[3] = pieces > 1 ? k * per_piece : 0; t6[4] = pieces > 1 ? min(T, (k + 1) * per_piece) : T;
    t6[5] = pieces > 1 ? s_slot0[c] + i : -1; t6[6] = s_tot[c]; t6[7] = (group * BM) & 63;
    if (pieces > 1 && k == 0) {
      int32_t* m = ml + (size_t)(s_merge0[c] + group) * 4;
      m[0] = r0; m[1] = rows; m[2] = s_slot0[c] + i; m[3] = pieces;
    }
  }
  if constexpr (DEAL) {
    lds_barrier();
    if (s_last) deal_lists(dl);
  }
}

// Query tiles beside the key lists: where the selection has left the lengths of the lists, one workgroup of a head plans its
// tiles while the others write its lists.  As a launch of its own behind them it took 5-6 us more (both sides with the smaller
// merge launch, below: 1 500 tokens 150 -> 148 us, 4 096 fp32 213 -> 208, 17 550 warm 1014 -> 1005, 32 760 with top-p 840 -> 828).
struct TilePlan {
  const int32_t* lengths; const int32_t* q_offs; int q_offs_stride;
  int maxtiles, BM, slots, allow_split;
  int32_t* tiles; int32_t* ntiles; int32_t* merge; int32_t* nmerge;
  Deal deal;
};

__device__ __forceinline__ void keys_of_list(int i, int h, int Cq, int cap, int maxr, int row_scale,
                            const int32_t* __restrict__ k_offs, int k_offs_stride,
                            const int32_t* __restrict__ k_count,
                            const int32_t* __restrict__ sel_idx, const int32_t* __restrict__ sel_cnt,
                            int32_t* __restrict__ rng_start, int32_t* __restrict__ rng_pre,
                            int32_t* __restrict__ rng_cnt, int32_t* __restrict__ krow, size_t kstride,
                            const int32_t* __restrict__ perm_k, int N) {
  const int tid = threadIdx.x;
  int32_t* rs = rng_start + ((size_t)h * Cq + i) * maxr;
  int32_t* rp = rng_pre + ((size_t)h * Cq + i) * (maxr + 1);
  constexpr int LR = 512;                  // ranges that LDS holds a copy of
  __shared__ int32_t l_rs[LR], l_rp[LR + 1];
  __shared__ int32_t s_nr, s_total;
  __shared__ int32_t s_we[4], s_wh[4], s_wlen[4], s_wst[4];
  {
    // The selected clusters in list order; a cluster whose rows follow the previous non-empty one's directly
    // extends its range.  256 entries per round: "end of the last non-empty entry before me" by a scan that
    // keeps the right operand when it is non-empty, then run starts and lengths by prefix sums; the state
    // after a round (last end, keys so far, ranges so far) is carried into the next.
    const int32_t* sel = sel_idx + ((size_t)h * Cq + i) * cap;
    const int cnt = min(sel_cnt[(size_t)h * Cq + i], cap);
    const int32_t* ko = k_offs + (size_t)h * k_offs_stride;
    const int kc = min(k_count[h], cap);                      // (a caller's count: the offsets end at the capacity)
    const int lane = tid & 63, wave = tid >> 6;
    int carry_e = -1, carry_total = 0, carry_nr = 0;          // identical in every thread
    for (int base = 0; base < cnt; base += 256) {
      const int t = base + tid;
      int sk = 0, ek = 0;
      bool valid = false;
      if (t < cnt) {
        const int j = sel[t];
        if (j >= 0 && j < kc) { sk = ko[j]; ek = ko[j + 1]; valid = ek > sk; }
      }
      const int len = valid ? ek - sk : 0;
      // inclusive scans inside the wave
      int ie = valid ? ek : -1, ih = valid ? 1 : 0, il = len;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const int oe = __shfl_up(ie, off), oh = __shfl_up(ih, off), ol = __shfl_up(il, off);
        if (lane >= off) { if (!ih) { ie = oe; ih = oh; } il += ol; }
      }
      if (lane == 63) { s_we[wave] = ie; s_wh[wave] = ih; s_wlen[wave] = il; }
      __syncthreads();
      // what precedes this thread: the carry, the earlier waves, the earlier lanes
      int pe = carry_e, ph = carry_e >= 0 ? 1 : 0, plen = carry_total;
      for (int w = 0; w < wave; ++w) { if (s_wh[w]) { pe = s_we[w]; ph = 1; } plen += s_wlen[w]; }
      const int le = __shfl_up(ie, 1), lh = __shfl_up(ih, 1);
      if (lane > 0 && lh) { pe = le; ph = 1; }
      plen += il - len;
      const bool start = valid && !(ph && pe == sk);
      int is = start ? 1 : 0;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) { const int o = __shfl_up(is, off); if (lane >= off) is += o; }
      if (lane == 63) s_wst[wave] = is;
      __syncthreads();
      int pst = carry_nr;
      for (int w = 0; w < wave; ++w) pst += s_wst[w];
      if (start) {
        const int r = pst + is - 1;
        rs[r] = sk; rp[r] = plen;
        if (r < LR) { l_rs[r] = sk; l_rp[r] = plen; }
      }
      // the carry of the next round, the same in every thread
      for (int w = 0; w < 4; ++w) { if (s_wh[w]) carry_e = s_we[w]; carry_total += s_wlen[w]; carry_nr += s_wst[w]; }
      __syncthreads();                         // the wave totals are free again
    }
    carry_total = min(carry_total, N);      // (a list that names clusters twice ends here: its row of krow holds N keys)
    if (tid == 0) {
      rp[carry_nr] = carry_total;
      rng_cnt[(size_t)h * Cq + i] = carry_nr;
      s_nr = carry_nr; s_total = carry_total;
    }
  }
  if (!krow) return;      // (the fp32 kernel finds its rows from the ranges: see attn_rows_listed)
  __syncthreads();        // the ranges are visible to the whole workgroup
  // Every key row of the concatenation, in order, as a byte offset (bf16) or a row number (fp32, row_scale 1): what
  // a key tile of the attention kernel loads its rows by.  Entries past the end (up to the padding the kernel may read ahead) repeat the
  // first row: they are loaded and never used.  A thread takes four entries in a row: one search (in LDS where the ranges
  // fit: its steps depend on one another), then the ranges one after the other, four rows asked for together and a 16-byte
  // store.  (With a search for every entry the searches bound it: 30 x 65 lists of 5 000 keys 28 us, now 21.)
  const int nr = s_nr, total = s_total;
  int32_t* kr = krow + ((size_t)h * Cq + i) * kstride;
  const int32_t* pk = perm_k + (size_t)h * N;      // sorted position -> token (rows stay where they are)
  const int padded = (total + 63) / 64 * 64 + KROW_PAD;
  auto fill = [&](const int32_t* srs, const int32_t* srp) __attribute__((always_inline)) {
    const int first = nr > 0 ? pk[srs[0]] * row_scale : 0;
    for (int p0 = 4 * tid; p0 < padded; p0 += 4 * 256) {
      int off[4] = {first, first, first, first};
      if (p0 < total) {
        int lo = 0, hi = nr - 1;                 // last range whose first position is <= p0
        while (lo < hi) { const int mid = (lo + hi + 1) >> 1; if (srp[mid] <= p0) lo = mid; else hi = mid - 1; }
        int shift = srs[lo] - srp[lo], next = lo + 1 < nr ? srp[lo + 1] : INT32_MAX, row[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int p = min(p0 + u, total - 1);
          if (p >= next) { ++lo; shift = srs[lo] - next; next = lo + 1 < nr ? srp[lo + 1] : INT32_MAX; }      // (every range has a key)
          row[u] = shift + p;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) { const int t = pk[row[u]] * row_scale; off[u] = p0 + u < total ? t : first; }
      }
      *reinterpret_cast<int4*>(kr + p0) = int4{off[0], off[1], off[2], off[3]};
    }
  };
  if (nr <= LR) fill(l_rs, l_rp); else fill(rs, rp);
}

template <bool TILES, bool DEAL>
__global__ __launch_bounds__(256, 8) void plan_sparse(int Cq, int cap, int maxr, int row_scale,
                            const int32_t* __restrict__ k_offs, int k_offs_stride,
                            const int32_t* __restrict__ k_count,
                            const int32_t* __restrict__ sel_idx, const int32_t* __restrict__ sel_cnt,
                            int32_t* __restrict__ rng_start, int32_t* __restrict__ rng_pre,
                            int32_t* __restrict__ rng_cnt, int32_t* __restrict__ krow, size_t kstride,
                            const int32_t* __restrict__ perm_k, int N, TilePlan tp) {
  const int h = blockIdx.x, i = (int)blockIdx.y - (TILES ? 1 : 0);      // (the workgroups that plan tiles, the longest chains, are the first)
  if (i >= 0) {
    keys_of_list(i, h, Cq, cap, maxr, row_scale, k_offs, k_offs_stride, k_count, sel_idx, sel_cnt, rng_start, rng_pre, rng_cnt, krow, kstride, perm_k, N);
    if (!TILES && tp.deal.planned && i == 0 && h == 0 && threadIdx.x == 0) *tp.deal.planned = 0;      // (for plan_tiles)
  } else if constexpr (TILES) {
    extern __shared__ int32_t plan_lds[];
    tiles_of_head<true, DEAL>(plan_lds, h, Cq, maxr, tp.maxtiles, tp.BM, tp.slots, tp.allow_split, tp.deal, tp.q_offs, tp.q_offs_stride, tp.lengths, nullptr, nullptr, tp.tiles,
                  tp.ntiles, tp.merge, tp.nmerge);
  }
}

template <bool DEAL>
__global__ __launch_bounds__(256) void plan_tiles(int Cq, int maxr, int maxtiles, int BM, int slots, int allow_split, Deal dl,
                                                  const int32_t* __restrict__ q_offs, int q_offs_stride,
                                                  const int32_t* __restrict__ rng_pre,
                                                  const int32_t* __restrict__ rng_cnt,
                                                  int32_t* __restrict__ tiles, int32_t* __restrict__ ntiles,
                                                  int32_t* __restrict__ merge, int32_t* __restrict__ nmerge) {
  constexpr int MAXC = DEAL ? PLAN_BESIDE : 4096;   // the largest q_clusters the library accepts
  __shared__ int32_t sm[plan_ints(MAXC, DEAL)];
  tiles_of_head<false, DEAL>(sm, blockIdx.x, min(Cq, MAXC), maxr, maxtiles, BM, slots, allow_split, dl, q_offs, q_offs_stride, nullptr, rng_pre, rng_cnt, tiles,
                ntiles, merge, nmerge);
}

// dense: one query "cluster" over all rows, one key range [0,N), in `pieces` chunks a query tile (attn_dense_shape)
__global__ void plan_dense(int N, int maxtiles, int BM, int pieces, int slots, int row_scale, int32_t* __restrict__ rng_start,
                           int32_t* __restrict__ rng_pre, int32_t* __restrict__ rng_cnt,
                           int32_t* __restrict__ tiles, int32_t* __restrict__ ntiles, int32_t* __restrict__ merge, int32_t* __restrict__ nmerge,
                           int32_t* __restrict__ krow, size_t kstride) {
  const int h = blockIdx.x;
  if (blockIdx.y > 0) {       // the other workgroups of a head fill its row-offset table (the identity)
    if (!krow) return;
    int32_t* kr = krow + (size_t)h * kstride;
    const int padded = (N + 63) / 64 * 64 + KROW_PAD;
    for (int p = (blockIdx.y - 1) * blockDim.x + threadIdx.x; p < padded; p += (gridDim.y - 1) * blockDim.x)
      kr[p] = p < N ? p * row_scale : 0;
    return;
  }
  if (threadIdx.x == 0) {
    rng_start[h] = 0; rng_pre[(size_t)h * 2] = 0; rng_pre[(size_t)h * 2 + 1] = N; rng_cnt[h] = 1;
    ntiles[h] = (N + BM - 1) / BM * pieces;
    nmerge[h] = pieces > 1 ? (N + BM - 1) / BM : 0;
  }
  int32_t* tl = tiles + (size_t)h * maxtiles * TILE_REC;
  const int T = (N + 63) / 64, per_piece = (T + pieces - 1) / pieces;
  for (int t = threadIdx.x; t / pieces * BM < N; t += blockDim.x) {
    const int group = t / pieces, k = t - group * pieces, r0 = group * BM, rows = min(BM, N - r0);
    int32_t* t6 = tl + (size_t)t * TILE_REC;
    t6[0] = 0; t6[1] = r0; t6[2] = rows; t6[3] = k * per_piece; t6[4] = min(T, (k + 1) * per_piece);
    t6[5] = pieces > 1 ? t : -1; t6[6] = N; t6[7] = r0 & 63;
    if (pieces > 1 && k == 0) {
      int32_t* m = merge + ((size_t)h * slots + group) * 4;
      m[0] = r0; m[1] = rows; m[2] = t; m[3] = pieces;
    }
  }
}

// Per-head figures of the last clustering and the last attention plan on this workspace: |C|, F, stages and
// |U| per stage from the Algorithm 1 state, and the (query, key) pairs the attention launch covers: executed
// = rows x keys of every query tile, issued = the same with rows rounded up to whole 32-query waves and keys
// to whole 64-key tiles (what the matrix cores are actually fed).
__global__ __launch_bounds__(256) void attn_stats(int Cq, int maxr, int maxtiles, const KState* __restrict__ st,
                                                  const int32_t* __restrict__ tiles, const int32_t* __restrict__ ntiles,
                                                  const int32_t* __restrict__ rng_pre, const int32_t* __restrict__ rng_cnt,
                                                  adacluster_head_stats* __restrict__ out) {
  const int h = blockIdx.x, tid = threadIdx.x;
  const int nt = min(ntiles[h], maxtiles);
  const int32_t* tl = tiles + (size_t)h * maxtiles * TILE_REC;
  long long ex = 0, is = 0;
  int whole = 0;                          // (fp32 tiles are counted per 64 rows)
  for (int t = tid; t < nt; t += 256) {
    const int32_t* t6 = tl + (size_t)t * TILE_REC;
    const int c = t6[0], rows = t6[2], kt0 = t6[3], kt1 = t6[4];
    const int total = rng_pre[((size_t)h * Cq + c) * (maxr + 1) + rng_cnt[(size_t)h * Cq + c]];
    const long long keys = max(0, min(total, kt1 * 64) - kt0 * 64);
    ex += (long long)rows * keys;
    is += (long long)((rows + 31) / 32 * 32) * ((keys + 63) / 64 * 64);
    whole += t6[7] == 0;
  }
  __shared__ long long s_ex[256], s_is[256];
  __shared__ int s_nt[256];
  s_ex[tid] = ex; s_is[tid] = is; s_nt[tid] = whole;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (tid < o) { s_ex[tid] += s_ex[tid + o]; s_is[tid] += s_is[tid + o]; s_nt[tid] += s_nt[tid + o]; }
    __syncthreads();
  }
  if (tid == 0) {
    adacluster_head_stats r;
    const KState& k = st[h];
    r.k_count = k.ccount; r.full_flag = k.full; r.stages = k.stage; r.q_tiles = s_nt[0];
    for (int i = 0; i <= ADACLUSTER_MAX_STAGES; ++i) r.unassigned[i] = i <= k.stage ? k.u_hist[i] : 0;
    r.reserved = 0;
    r.executed_pairs = s_ex[0]; r.issued_pairs = s_is[0];
    out[h] = r;
  }
}

int launch_attn_stats(hipStream_t s, int H, int Cq, int maxr, int maxtiles, const KState* st, const int32_t* tiles,
                      const int32_t* ntiles, const int32_t* rng_pre, const int32_t* rng_cnt, adacluster_head_stats* out) {
  attn_stats<<<H, 256, 0, s>>>(Cq, maxr, maxtiles, st, tiles, ntiles, rng_pre, rng_cnt, out);
  return hipGetLastError() == hipSuccess ? 0 : ADACLUSTER_E_INTERNAL;
}

struct AttnArgs {
  const void* Q; const void* K; const void* V; void* O;
  const int32_t* perm_q;        // sorted query position -> token (NULL: identity)
  const int32_t* tiles; const int32_t* ntiles;
  int H, N, Cq, maxtiles;
  float scale_log2e;            // softmax scale x log2(e)
  int head_major;               // workgroup -> (head, tile) mapping, see attn_mfma
  float* part_o; float* part_ml;   // partial slots of cut key lists: [H][slots][BM][d], [H][slots][BM][2]
  int slots, BM;
  const int32_t* krow; size_t kstride;   // every key row of a query cluster's list (byte offset, fp32: row number): [H][Cq][kstride]
  const int32_t* rng_start; const int32_t* rng_pre; const int32_t* rng_cnt; int maxr;   // the ranges it was written from, and
  const int32_t* perm_k;                 // their order -> token (NULL: identity): for the fp32 kernel without a table
  int splits;                            // fp32: most pieces a key list may go in, and what f32_pieces() says
  Pieces pieces;
  const int32_t* deal; int deal_stride;  // tiles dealt by work (Deal::lists; NULL: not)
};

// Workgroup -> (head, query tile) of a launch of pick_tile_grid.  Workgroups go to the 8 XCDs round-robin in launch order,
// each with its own L2, so XCD = blockIdx.x % 8 and blockIdx.x / 8 is a slot in that XCD's own list of tiles: of every
// head, in head order, the XCD takes a contiguous eighth (the tiles of one query cluster stream the same K/V rows, and so
// do it behind the same L2).
// Only the device knows how many tiles a head has.  Up to PICK_HEADS heads the list is cut from those counts here, so that
// the workgroups without work are the last of the grid.  (With a grid row per head, sized for the most tiles a head
// could have, there are empty ones between the heads, and each takes its turn on a CU.)  More heads have a grid row each:
// the search costs a trip to memory per 64 heads, and past 2^32 threads a grid dimension ends.  Calls of 70, 150 and 256
// heads of 2 000 rows, d=64, 33 clusters 288, 579 and 975 us by search, 331, 664 and 1 107 by rows; of 1 000 rows and 200 clusters
// 228, 456, 802 and 216, 417, 704; 1 024 heads of 128 rows 718 by rows (by search, when tiles were 64 rows, 1 625).
// With `splits` > 1 the key lists of the tiles that would not fill the chip once more are split: an XCD runs `resident`
// workgroups at a time, and the tiles past the last whole round of them (all of them in a small launch) go in pieces (z says
// which; f32_pieces() how many), so that no CU is left with a whole one when the others are done.  585 tiles, d=128, are 75
// an XCD that holds 64 workgroups: 64 whole and 11 in four pieces, 198 us; all of them in two pieces, three rounds, 222.
// Returns false where the list has ended.

__device__ __forceinline__ bool pick_tile(const int32_t* __restrict__ ntiles, int H, const Pieces& pieces, int splits, int resident, int& h, int& tile,
                                          int& z, int& sp) {
  const int xcd = blockIdx.x & 7, lane = threadIdx.x & 63;
  int slot = blockIdx.x >> 3;
  z = 0; sp = 1;
  if (H > PICK_HEADS) {
    h = blockIdx.y;
    const int nt = ntiles[h], w = (nt + 7) >> 3;
    tile = xcd * w + slot;
    return slot < w && tile < nt;
  }
  int nt, w, incl;                                         // 64 heads at a time, one per lane: tiles, this XCD's share of them
  auto take = [&](int h0) __attribute__((always_inline)) { // (the last XCD's may be short), and the shares up to here
    nt = h0 + lane < H ? ntiles[h0 + lane] : 0;
    w = (nt + 7) >> 3;
    incl = w;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) { const int v = __shfl_up(incl, o); if (lane >= o) incl += v; }
  };
  take(0);
  if (splits > 1) {
    int total = __builtin_amdgcn_readlane(incl, 63);
    for (int h0 = 64; h0 < H; h0 += 64) { take(h0); total += __builtin_amdgcn_readlane(incl, 63); }
    if (H > 64) take(0);
    const int rest = total % resident, whole = total - rest;
    if (slot >= whole) {
      if (rest == 0) return false;
      sp = pieces_of(pieces, rest);
      z = (slot - whole) / rest;                           // (first pieces first: short lists have no others, which end at once)
      if (z >= sp) return false;
      slot -= z * rest;
    }
  }
  int base = 0;
  for (int h0 = 0; h0 < H; h0 += 64) {
    if (h0 > 0) take(h0);
    const uint64_t past = __ballot(base + incl > slot);
    if (past) {
      const int l = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)past) - 1);
      const int wl = __builtin_amdgcn_readlane(w, l);
      h = h0 + l;
      tile = xcd * wl + slot - base - __builtin_amdgcn_readlane(incl, l) + wl;
      return tile < __builtin_amdgcn_readlane(nt, l);
    }
    base += __builtin_amdgcn_readlane(incl, 63);
  }
  return false;
}

// ------------------------------------------------------------------------------------------
// bf16 MFMA kernel
// ------------------------------------------------------------------------------------------
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4_t;
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;
typedef __attribute__((address_space(3))) void lds_void_t;

// LDS transpose read (16-bit elements): inside each group of 16 lanes, lane r supplies the address
// of 4 consecutive elements and lane i receives element i%4 of the rows addressed by lanes
// i/4, i/4+4, i/4+8, i/4+12.
__device__ __forceinline__ s16x4_t lds_read_tr16(const char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)p);
}

// One workgroup = NW waves of 32 queries each; all waves share 64-key K and V tiles.  Tiles go global -> LDS
// directly (no register staging) as 16-byte chunks into a ring of NBUF stages, NBUF-1 tiles ahead of the
// arithmetic, one barrier per tile.  A tile row is unpadded and its 16-byte chunks are permuted by a row-dependent
// XOR that keeps the operand reads of either tile free of bank conflicts (see swz_k, swz_v).  The rows of a tile come
// from the row-offset table plan_sparse / plan_dense wrote: its 64 entries for a tile are themselves loaded
// global -> LDS, 2*(NBUF-1) tiles ahead, so that no wave walks a range list and no load waits on a register.
// LDS layout: [row offsets: NBUF x 64][K ring: NBUF tiles][V ring: NBUF tiles]; with the K tiles (and the V
// tiles) side by side, a stage is reached from one set of address registers by an immediate offset (< 64 KB;
// the start of the V ring is part of the V address registers).
template <int D, int NW, int NBUF, int MINB, int VPRE>
__global__ __launch_bounds__(NW * 64, MINB) void attn_mfma(AttnArgs a) {
  constexpr int BN = 64, NT = NW * 64, KS = D / 16, DB = D / 32, CH = D / 8, ROWB = D * 2;
  constexpr int ITEMS = BN * CH, PT = ITEMS / NT, TILEB = BN * ROWB, PD = NBUF - 1;
  constexpr int VM_STEP = 2 * PT + 1;             // vector-memory operations a wave issues per tile
  constexpr int ISSUE_J0 = D == 128 ? 2 : 3, ISSUE_STRIDE = (2 * KS - ISSUE_J0) / VM_STEP;     // the requests spread over the S products
  static_assert(ISSUE_STRIDE >= 1, "more requests than S products to put them behind");
  constexpr int RIDXB = NBUF * BN * 4;            // bytes of the row-offset slots at the start of LDS
  constexpr int KRING = NBUF * TILEB;             // bytes of the ring of K tiles (the ring of V tiles follows it)
  static_assert(ITEMS % NT == 0, "tile chunks must divide evenly over the threads");
  static_assert(NBUF == 2 || NBUF == 4, "two or four stages");
  static_assert(2 * PD + 1 <= KROW_PAD / 64, "the row-offset table is padded for the read-ahead");
  static_assert(64 % NW == 0, "every wave loads an equal share of a tile's row offsets");

  // Workgroups go to the 8 XCDs round-robin in launch order (gridDim.x is a multiple of 8, so
  // XCD = blockIdx.x % 8), and each XCD has its own L2.
  int h, tile;
  if (a.deal) {
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int32_t* list = a.deal + (size_t)xcd * a.deal_stride;
    const int e = list[DEAL_HEAD + slot];          // (asked for with the head of the list)
    if (slot >= list[0]) return;
    const DealtTile dt = dealt_tile(e);
    h = dt.h; tile = dt.tile;
  } else if (a.head_major) {
    // Heads are dealt to XCDs whole, eight at a time: all query tiles of a head then stream that
    // head's K/V rows behind one L2.  The H % 8 heads left over are split eight ways by tile.
    const int gx = gridDim.x, gx8 = gx >> 3;
    const int xcd = blockIdx.x & 7, slot = (blockIdx.y * gx + blockIdx.x) >> 3;
    const int Hfull = (gridDim.y >> 3) << 3, full_slots = (Hfull >> 3) * gx;
    if (slot < full_slots) {
      h = (slot / gx) * 8 + xcd; tile = slot % gx;
      if (tile >= a.ntiles[h]) return;
    } else {
      const int r = slot - full_slots, j = r % gx8;
      h = Hfull + r / gx8;
      const int nt = a.ntiles[h], per = (nt + 7) >> 3;    // eighths of the tiles the head has, not of the grid
      tile = xcd * per + j;
      if (j >= per || tile >= nt) return;
    }
  } else {
    // Every head is split eight ways: an XCD takes a contiguous run of its query tiles (the tiles
    // of one query cluster stream the same K/V rows, and so do it behind the same L2).  The runs
    // are eighths of the tiles the head has; the grid is sized for the most it could have.
    h = blockIdx.y;
    const int nt = a.ntiles[h], per = (nt + 7) >> 3, j = blockIdx.x >> 3;
    tile = (blockIdx.x & 7) * per + j;
    if (j >= per || tile >= nt) return;
  }
  const int32_t* tl = a.tiles + ((size_t)h * a.maxtiles + tile) * TILE_REC;
  const int qc = tl[0], row0 = tl[1], nrows = tl[2];
  const int kt0 = tl[3], kt1 = tl[4], pslot = tl[5];    // this workgroup's share of the key list
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 31, hb = lane >> 5;

  // positions below are relative to the first key of the share
  const int pbase = kt0 * BN;
  const int total = max(0, min(tl[6], kt1 * BN) - pbase);     // (tl[6]: keys of the whole list; two dependent loads fewer than from the ranges)
  const int T = (total + BN - 1) / BN;
  const int32_t* krow = a.krow + ((size_t)h * a.Cq + qc) * a.kstride + pbase;   // byte offsets of the key rows

  const bf16raw* Qh = (const bf16raw*)a.Q + (size_t)h * a.N * D;
  const char* Kh = (const char*)a.K + (size_t)h * a.N * ROWB;
  const char* Vh = (const char*)a.V + (size_t)h * a.N * ROWB;
  bf16raw* Oh = (bf16raw*)a.O + (size_t)h * a.N * D;
  const int32_t* pq = a.perm_q ? a.perm_q + (size_t)h * a.N : nullptr;

  // query token of this lane and the B operand of S
  int qtok = -1;
  bf16x8_t qf[KS];
  const bool wave_has_rows = wave * 32 < nrows;
  {
    const int rr = wave * 32 + c;
    if (rr < nrows) qtok = pq ? pq[row0 + rr] : row0 + rr;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      uint4 raw = {0, 0, 0, 0};
      if (qtok >= 0) raw = *reinterpret_cast<const uint4*>(Qh + (size_t)qtok * D + ks * 16 + hb * 8);
      qf[ks] = *reinterpret_cast<const bf16x8_t*>(&raw);
    }
  }

  f32x16_t oacc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) oacc[db][v] = 0.f;
  // Soft-max state of this lane's query: probabilities are taken relative to a reference mref that is only
  // moved when it has to be (see soft-max below); lrun is the sum of the probabilities so far.  The reference starts at
  // the lowest value that is finite when scaled too: every score above -inf is far enough above it to move it, and tiles
  // of -inf alone, at the start of the share or all through it, leave it there with a sum and an accumulator of zero (from
  // -inf they would make both NaN, and the launch of small dense calls, whose shares start anywhere in a list, with them).
  float mref = -3.402823466e38f / fmaxf(a.scale_log2e, 1.f), lrun = 0.f;

  // Where a 16-byte chunk sits inside its (unpadded) tile row: chunk q of row r is in slot q ^ swz(r).  A row
  // is 256 B (d=128: every row starts at bank 0) or 128 B (d=64: rows two apart do), so the slot alone decides
  // the banks, and the two tiles are read in different shapes:
  //   K: a 16-byte operand read takes the same chunk of 16 consecutive rows per cycle -> 16 distinct slots
  //      (d=128), or 8 slots x the two row parities (d=64);
  //   V: a transpose read takes 64 contiguous bytes (4 slots) of 4 consecutive rows per cycle -> the rows
  //      must differ in the slot's upper bits; rows 8 apart share a swizzle, so the second half of an operand
  //      is a constant offset away.
  // Measured on the LDS alone: 3.7 and 2.2 cycles per read against 7.5 and 7.5 (3.9 at d=64) with q ^ (r & 7).
  auto swz_k = [](int r) __attribute__((always_inline)) { return D == 128 ? (r & 15) : ((r >> 1) & 7); };
  auto swz_v = [](int r) __attribute__((always_inline)) { return D == 128 ? ((r & 3) << 2) : (((r >> 1) & 1) << 2); };
  // thread -> (row, slot) of its PT chunks of a tile, and the global chunk that slot holds in either tile
  int lrow[PT], lswz_k[PT], lswz_v[PT];
#pragma unroll
  for (int i = 0; i < PT; ++i) {
    const int item = tid + i * NT;
    lrow[i] = item / CH;
    lswz_k[i] = ((item % CH) ^ swz_k(lrow[i])) * 16;
    lswz_v[i] = ((item % CH) ^ swz_v(lrow[i])) * 16;
  }
  __shared__ __attribute__((aligned(16))) char lds[RIDXB + 2 * KRING];
  char* const ldk = lds + RIDXB;                  // the K ring (compute_tile's V addresses carry KRING themselves)
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void_t*)lds;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  // the 64 row offsets of tile t go to the offsets slot of stage `st`, an equal share per wave
  const uint32_t ridx_voff = (uint32_t)((wave_u * (BN / NW) + (lane % (BN / NW))) * 4);
  auto issue_ridx = [&](int st, int t) __attribute__((always_inline)) {
    if (lane < BN / NW)
      dma_b32(lds0 + st * (BN * 4) + wave_u * (BN / NW) * 4, ridx_voff, krow + (size_t)t * BN);
  };
  auto issue_tile_op = [&](int st, const int32_t* off, int n) __attribute__((always_inline)) {     // operation n of issue_tile
    const int i = n >> 1;
    const uint32_t dst = lds0 + RIDXB + st * TILEB + (wave_u * 64 + i * NT) * 16;
    if ((n & 1) == 0) dma_b128(dst, (uint32_t)off[i] + (uint32_t)lswz_k[i], Kh);
    else dma_b128(dst + KRING, (uint32_t)off[i] + (uint32_t)lswz_v[i], Vh);
  };
  auto issue_tile = [&](int st, const int32_t* off) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const uint32_t dst = lds0 + RIDXB + st * TILEB + (wave_u * 64 + i * NT) * 16;     // wave-uniform; the lane offset is implicit
      dma_b128(dst, (uint32_t)off[i] + (uint32_t)lswz_k[i], Kh);
      dma_b128(dst + KRING, (uint32_t)off[i] + (uint32_t)lswz_v[i], Vh);
    }
  };

  // operand addresses inside a tile (bytes), fixed for the whole kernel
  int kaddr[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) kaddr[ks] = c * ROWB + (((ks * 2 + hb) ^ swz_k(c)) * 16);
  // The 8 accumulator values a lane feeds to one P V step are keys 4*hb + {0..3} and
  // 8 + 4*hb + {0..3} of a 16-key group; the V operand is gathered to match by two transpose
  // reads: this lane addresses key 4*hb + (lane%16)/4, columns 16*((lane/16)%2) + 4*(lane%4) .. +3
  // and receives column lane%32 of the four keys.
  int vaddr[DB];
  {
    const int i16 = lane & 15, blk = lane >> 4;
    const int vrow = 4 * hb + (i16 >> 2);
    const int gl = 2 * (blk & 1) + ((i16 & 3) >> 1);
#pragma unroll
    for (int db = 0; db < DB; ++db) vaddr[db] = KRING + vrow * ROWB + (((db * 4 + gl) ^ swz_v(vrow)) * 16) + 8 * (i16 & 1);
  }       // (the offset of the V ring sits in the register: what an LDS read adds as an immediate must stay below 64 KB)
  const bf16x2_t ones2 = {(__bf16)1.0f, (__bf16)1.0f};   // row sums use the rounded probabilities P V uses
  const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const float sc = a.scale_log2e;
  constexpr float P_LIMIT = 65536.f;      // a tile whose probabilities sum past this moves the reference

  // `prep` and `issue(n)`, n < ND: the requests of the tiles further ahead (row offsets out of LDS, then ND
  // direct-to-LDS loads), placed by compute_tile where they cost nothing: the offsets are read behind the K
  // operands, the loads are issued one by one between the S products, in the shadow of the matrix pipe.
  auto compute_tile = [&](const char* ks_, const char* vs_, int nvalid /* < BN only on a masked tail tile */,
                          auto masked, auto&& prep, auto&& issue, auto nd_) __attribute__((always_inline)) {
    constexpr bool MASK = decltype(masked)::value;
    constexpr int ND = decltype(nd_)::value;
    // All K operands of the tile are requested before the first product, and (below) the V operands before
    // the soft-max arithmetic: an LDS read takes a hundred cycles or more to come back, and the compiler, left
    // alone, requests an operand only one product ahead of its use.  The empty asm statements are fences for
    // memory operations (reads do not sink below them); the scheduling barrier behind each keeps the products
    // from rising above the reads that follow their own operands' (a product placed between two reads makes the
    // wave wait for its operand before the next read is even requested: measured, 5 % of the kernel at d=64).
    f32x16_t sacc[2];
    bf16x8_t ka[2][KS];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        ka[kb][ks] = *reinterpret_cast<const bf16x8_t*>(ks_ + kb * 32 * ROWB + kaddr[ks]);
    asm volatile("" ::: "memory");
    prep();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        sacc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[kb][ks], qf[ks], ks == 0 ? zero16 : sacc[kb], 0, 0, 0);
        // request n goes behind product ISSUE_J0 + n * ISSUE_STRIDE
        const int j = kb * KS + ks;
        if (ND > 0 && j >= ISSUE_J0 && (j - ISSUE_J0) % ISSUE_STRIDE == 0 && (j - ISSUE_J0) / ISSUE_STRIDE < ND) {
          __builtin_amdgcn_sched_barrier(0);
          issue((j - ISSUE_J0) / ISSUE_STRIDE);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    static_assert(ND == 0 || ISSUE_J0 + (ND - 1) * ISSUE_STRIDE < 2 * KS, "every request finds a product to go behind");
    bf16x8_t va[VPRE > 0 ? VPRE : 1][2][2];
#pragma unroll
    for (int db = 0; db < VPRE; ++db)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          const char* vp = vs_ + (kb * 32 + 16 * s2) * ROWB + vaddr[db];
          const s16x4_t lo = lds_read_tr16(vp), hi = lds_read_tr16(vp + 8 * ROWB);
          const s16x4_t both[2] = {lo, hi};
          va[db][kb][s2] = *reinterpret_cast<const bf16x8_t*>(both);
        }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    // accumulator value v of block kb is key  kb*32 + 8*(v/4) + 4*hb + v%4
    if (MASK) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int key = kb * 32 + 8 * (v >> 2) + 4 * hb + (v & 3);
          if (key >= nvalid) sacc[kb][v] = -INFINITY;
        }
    }
    // Soft-max.  p = 2^((s - mref) scale): any reference gives the same normalised result as long as nothing
    // overflows, so no maximum is taken per tile.  The row sum of the tile tells when the reference is too
    // low (on the first tile with a score above -inf the sum is +inf): only then is the tile's maximum taken,
    // the reference moved up to it and the accumulator rescaled.
    bf16x8_t pf[2][2];
    float rsum;
    auto probabilities = [&]() __attribute__((always_inline)) {
      const float moff = mref * sc;
      float part[2][2];                    // four chains of sums, so that an add does not wait for the one before it
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          uint32_t w[4];
          part[kb][s2] = 0.f;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float p0 = __builtin_amdgcn_exp2f(fmaf(sacc[kb][8 * s2 + 2 * j], sc, -moff));
            const float p1 = __builtin_amdgcn_exp2f(fmaf(sacc[kb][8 * s2 + 2 * j + 1], sc, -moff));
            w[j] = pack_bf16x2(p0, p1);
            part[kb][s2] = __builtin_amdgcn_fdot2_f32_bf16(*reinterpret_cast<const bf16x2_t*>(&w[j]), ones2, part[kb][s2], false);
          }
          const uint4 pk = {w[0], w[1], w[2], w[3]};
          pf[kb][s2] = *reinterpret_cast<const bf16x8_t*>(&pk);
        }
      rsum = (part[0][0] + part[0][1]) + (part[1][0] + part[1][1]);
    };
    probabilities();
    if (__any(!(rsum <= P_LIMIT))) {
      float tmax = sacc[0][0];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v) tmax = fmaxf(tmax, sacc[kb][v]);
      tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
      const float mnew = fmaxf(mref, tmax);
      const float alpha = __builtin_amdgcn_exp2f((mref - mnew) * sc);
      mref = mnew;
      lrun *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[db][v] *= alpha;
      probabilities();
    }
    lrun += rsum;
    asm volatile("" ::: "memory");          // the V operands that were not requested ahead are requested from here on,
    bf16x8_t vb[DB - VPRE > 0 ? DB - VPRE : 1][2][2];      // ALL of them before the first product (second fence): left
#pragma unroll                                            // alone, the compiler requests an operand one product ahead
    for (int db = VPRE; db < DB; ++db)                     // of its use and every product then waits out an LDS read
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          const char* vp = vs_ + (kb * 32 + 16 * s2) * ROWB + vaddr[db];
          const s16x4_t lo = lds_read_tr16(vp), hi = lds_read_tr16(vp + 8 * ROWB);
          const s16x4_t both[2] = {lo, hi};
          vb[db - VPRE][kb][s2] = *reinterpret_cast<const bf16x8_t*>(both);
        }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int db = 0; db < DB; ++db) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
          oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(db < VPRE ? va[db < VPRE ? db : 0][kb][s2] : vb[db >= VPRE ? db - VPRE : 0][kb][s2],
                                                             pf[kb][s2], oacc[db], 0, 0, 0);
    }
  };

  // Tile t lives in stage t % NBUF; the row offsets of tile t sit in the offsets slot of stage (t + 1) % NBUF,
  // the stage whose tile is being worked on when the loads of tile t are issued.  In step t:
  //   loads of tile t + PD          -> stage (t + PD) % NBUF (free since step t - 1), rows from the offsets slot
  //                                    of stage t % NBUF
  //   row offsets of tile t + 2 PD  -> the offsets slot of stage (t + PD) % NBUF
  //   arithmetic of tile t
  //   wait until this wave's loads of tile t + 1 have landed, barrier.
  // Loads are issued for tiles past the end too (the table is padded), so that the number of operations in
  // flight is the same in every step and one constant serves the wait.
  auto step = [&](auto stage, int t) __attribute__((always_inline)) {
    constexpr int U = decltype(stage)::value, G = (U + PD) % NBUF;
    int32_t off[PT];
    auto prep = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < PT; ++i) off[i] = reinterpret_cast<const int32_t*>(lds + U * (BN * 4))[lrow[i]];
    };
    auto issue = [&](int n) __attribute__((always_inline)) {
      if (n < 2 * PT) issue_tile_op(G, off, n); else issue_ridx(G, t + 2 * PD);
    };
    if (wave_has_rows) {
      compute_tile(ldk + U * TILEB, ldk + U * TILEB, BN, std::false_type{}, prep, issue, std::integral_constant<int, VM_STEP>{});
    } else {               // a wave without query rows still loads its share of the tiles
      prep();
#pragma unroll
      for (int n = 0; n < VM_STEP; ++n) issue(n);
    }
    wait_vmcnt<(PD - 1) * VM_STEP>();
    lds_barrier();
  };

  const int Tlast = T - 1;       // the loop takes tiles 0 .. Tlast-1; the last one, full or ragged, is peeled
  if (T > 0) {
    // tiles 0 .. PD-1: rows straight from the table; row offsets of tiles PD .. 2 PD - 1 to their slots
#pragma unroll
    for (int t = 0; t < PD; ++t) {
      int32_t off[PT];
#pragma unroll
      for (int i = 0; i < PT; ++i) off[i] = krow[(size_t)t * BN + lrow[i]];
      issue_tile(t, off);
    }
#pragma unroll
    for (int t = PD; t < 2 * PD; ++t) issue_ridx((t + 1) % NBUF, t);
    wait_vmcnt<0>();
    lds_barrier();
    if constexpr (NBUF == 2) {
      for (int t = 0; t < Tlast; t += 2) {
        step(std::integral_constant<int, 0>{}, t);
        if (t + 1 >= Tlast) break;
        step(std::integral_constant<int, 1>{}, t + 1);
      }
    } else {
      for (int t = 0; t < Tlast; t += 4) {
        step(std::integral_constant<int, 0>{}, t);
        if (t + 1 >= Tlast) break;
        step(std::integral_constant<int, 1>{}, t + 1);
        if (t + 2 >= Tlast) break;
        step(std::integral_constant<int, 2>{}, t + 2);
        if (t + 3 >= Tlast) break;
        step(std::integral_constant<int, 3>{}, t + 3);
      }
    }
    wait_vmcnt<0>();       // nothing of this wave is still on its way to LDS when it ends
    const int u = Tlast % NBUF;
    if (wave_has_rows) compute_tile(ldk + u * TILEB, ldk + u * TILEB, total - Tlast * BN, std::true_type{}, [] {}, [](int) {},
                                    std::integral_constant<int, 0>{});
  }

  // O^T accumulator value v of block db is column  db*32 + 8*(v/4) + 4*hb + v%4  of query c
  {
    const float l = lrun + __shfl_xor(lrun, 32);
    if (pslot >= 0) {
      // a chunk of a cut key list: leave the unnormalised accumulator, the reference and the
      // row sum in this chunk's slot; attn_merge combines the chunks of the query tile
      const int rr = wave * 32 + c;
      const size_t so = ((size_t)h * a.slots + pslot) * a.BM + rr;
      float* po = a.part_o + so * D;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float4 o = {oacc[db][4 * i], oacc[db][4 * i + 1], oacc[db][4 * i + 2], oacc[db][4 * i + 3]};
          *reinterpret_cast<float4*>(po + db * 32 + 8 * i + 4 * hb) = o;
        }
      if (hb == 0) { a.part_ml[so * 2] = mref; a.part_ml[so * 2 + 1] = l; }
      return;
    }
    const float inv = l > 0.f ? 1.0f / l : total > 0 ? NAN : 0.f;      // (no key: zero; no score above -inf: NaN, as 0 / 0)
    if (qtok < 0) return;
    bf16raw* orow = Oh + (size_t)qtok * D;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint2 o;
        o.x = pack_bf16x2(oacc[db][4 * i] * inv, oacc[db][4 * i + 1] * inv);
        o.y = pack_bf16x2(oacc[db][4 * i + 2] * inv, oacc[db][4 * i + 3] * inv);
        *reinterpret_cast<uint2*>(orow + db * 32 + 8 * i + 4 * hb) = o;
      }
  }
}

// ------------------------------------------------------------------------------------------
// fp32 kernel (the accuracy path of fp32 inputs): the same S^T = K Q^T / O^T += V^T P^T walk on the
// matrix cores with v_mfma_f32_32x32x2_f32 (fp32 products, fp32 accumulation)
// ------------------------------------------------------------------------------------------
// A workgroup is a query tile of 32 queries; its four waves take every fourth 32-key tile of the key list, each
// with an accumulator and soft-max state of its own, and meet once at the end.  In the 32x32 accumulator a lane
// (c = lane % 32, hb = lane / 32) owns query c and the keys 8*(v/4) + 4*hb + v%4 of the tile, v = 0..15.  The
// two values a lane pair supplies per product step may be any pair of the contraction index as long as both
// operands agree: for S step 4*i + j the pair is (dim 8*i + j, dim 8*i + 4 + j), so that a lane takes a 16-byte piece of
// its row for four steps; for P V step j contracts exactly the keys of accumulator value j, so the probabilities
// are the B operand as they stand, and the A operand takes the columns c*DB .. +DB-1 of a V row per lane (column
// block db of the accumulator is then the columns i*DB + db), one coalesced vector load a key and no LDS.
// K tiles go global -> LDS directly into an area of the wave's own, row by row (loaded straight into registers a
// lane would have to fetch its own row, 64 lines per load): the next tile is requested in the middle of the P V
// products; V rows are requested around the S products.  No barrier inside the loop.
// Slot s (16 bytes) of row r holds piece s ^ (r & 15): the operand reads of 16 consecutive rows hit 16 bank groups.
// What bounds the path: the fp32 matrix rate (a product of 32x32x2 holds the pipe for 64 cycles) once there are
// workgroups enough, which is why the key list is split: over the waves, and where the launch is small (4 096
// queries are 128 tiles for 256 CUs) over up to four workgroups as well, which leave unnormalised partial results
// that attn_merge_f32 combines (see pick_tile), lists too short for that aside.  Vector instructions do not run under an fp32 product on this chip
// (the co-execution counter reads 0), so every one of them adds its four cycles: the masks are for the last tile
// only, the accumulator is rescaled only when the maximum has moved, and addresses inside a head are 32-bit offsets.
// Without these the 545 vector instructions a tile took a fifth of the time.
// LISTED: the key rows of a tile come from the table of the planning step, and a head has less than 4 GiB; else they are
// searched in the ranges of the list, tile by tile, and offsets are 64-bit (attn_rows_listed says which).
// Measured against a kernel of two waves of 32 queries a workgroup with K and V through LDS and three barriers a tile
// (kernel and merge): dense, d=128, 4 heads x 8 192 rows 75 -> 125 TFLOP/s (of 154 that an fp32 GEMM reaches), 1 x 4 096
// 10 -> 104; one head of 4 096 queries (d=64) against a quarter of its keys 132 -> 28 us, three of 5 007 (d=128) against a
// third 405 -> 197 us, six of 5 000 (d=64) against 57 keys 23 -> 22 us.  (Eight waves a workgroup, one workgroup a CU: a sixth
// slower at 4 096.)  At d=64 three workgroups a CU (168 registers; at 172 two: 150 heads of 1 000 rows 319 and 400 us).
template <int D, bool LISTED>
__global__ __launch_bounds__(F32_WAVES * 64, D == 64 ? 3 : 2) void attn_f32(AttnArgs a) {
  constexpr int BN = 32, DB = D / 32, NW = F32_WAVES, SROW = D + 4, PPR = D / 4, RPI = 64 / PPR;   // 16-byte pieces a row, rows a load
  int h, tile, z, sp;
  if (a.deal) {
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int32_t* list = a.deal + (size_t)xcd * a.deal_stride;
    const int e = list[DEAL_HEAD + slot];
    if (slot >= list[0]) return;
    const DealtTile dt = dealt_tile(e);
    h = dt.h; tile = dt.tile; z = dt.z; sp = dt.sp;
  } else if (!pick_tile(a.ntiles, a.H, a.pieces, a.splits, f32_resident(D), h, tile, z, sp)) return;
  const int32_t* tl = a.tiles + ((size_t)h * a.maxtiles + tile) * TILE_REC;          // (key lists are never cut for fp32)
  const int qc = tl[0], row0 = tl[1], nrows = tl[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 31, hb = lane >> 5;
  const int total = tl[6], T = (total + BN - 1) / BN;
  // The workgroups that share this list: not more than its tiles give work to, the others end here.  A list of a single one
  // is written out by it.
  const int splits = min(sp, max(1, (T + NW - 1) / NW));
  if (z >= splits) return;
  const int32_t* kr = a.krow + ((size_t)h * a.Cq + qc) * a.kstride;           // key rows of the list, in order
  const float* Qh = (const float*)a.Q + (size_t)h * a.N * D;
  const char* Kh = (const char*)((const float*)a.K + (size_t)h * a.N * D);
  const char* Vh = (const char*)((const float*)a.V + (size_t)h * a.N * D);
  typedef typename std::conditional<LISTED, uint32_t, size_t>::type off_t;
  // a wave's K tile in the loop; after it, its accumulator, a (padded) row per query
  __shared__ __attribute__((aligned(16))) float sk[NW * 32 * SROW];
  __shared__ float sm[NW][32], sl[NW][32];
  char* const kt = reinterpret_cast<char*>(sk) + __builtin_amdgcn_readfirstlane(wave) * (BN * D * 4);
  const uint32_t kt_lds = (uint32_t)(uintptr_t)(lds_void_t*)kt;
  const int32_t* pq = a.perm_q ? a.perm_q + (size_t)h * a.N : nullptr;
  // The addresses of a tile are worked out anew for every tile (the empty asm statements hide that they do not
  // change): hoisted out of the loop they would take 50 registers that are not there.
  auto issue_k = [&](int idx) __attribute__((always_inline)) {                // idx: row number of key c, in every lane
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int lr = ln / PPR, lp = ln % PPR;                // row and piece of the RPI rows that one direct load brings
#pragma unroll
    for (int n = 0; n < BN / RPI; ++n) {
      const int row = __builtin_amdgcn_ds_bpermute(lr * 4 + n * RPI * 4, idx);
      const uint32_t piece = (uint32_t)(lp ^ ((n * RPI + lr) & 15)) * 16;
      const off_t off = (off_t)(uint32_t)row * (D * 4) + piece;
      if constexpr (LISTED) dma_b128(kt_lds + n * 1024, off, Kh);
      else dma_b128(kt_lds + n * 1024, Kh + off);
    }
  };
  // Row number of key c of tile t, for a wave's tiles in order.  Without the table: r0 is a range that starts at or before
  // the tile, b the starts of the 64 ranges behind it, one a lane; once at most 32 of them lie before the tile, its keys are
  // in those ranges (every range has a key), and each lane counts the starts up to its own.
  int r0 = 0;
  auto key_row = [&](int t) __attribute__((always_inline)) {
    if constexpr (LISTED) return kr[t * BN + c];
    const size_t list = (size_t)h * a.Cq + qc;
    const int32_t* rs = a.rng_start + list * a.maxr;
    const int32_t* rp = a.rng_pre + list * (a.maxr + 1);
    const int nr = a.rng_cnt[list], p = min(t * BN + c, total - 1);          // (keys past the end repeat the last: masked)
    int b;
    for (;;) {
      b = r0 + 1 + lane < nr ? rp[r0 + 1 + lane] : INT32_MAX;
      const int before = __popcll(__ballot(b <= t * BN));
      if (before <= 32) break;
      r0 += before;
    }
    int n = 0;
#pragma unroll
    for (int step = 32; step; step >>= 1)
      if (__builtin_amdgcn_ds_bpermute((n + step - 1) * 4, b) <= p) n += step;
    const int row = rs[r0 + n] + p - rp[r0 + n];
    return a.perm_k ? a.perm_k[(size_t)h * a.N + row] : row;
  };
  // (the table is padded: entries past the list are rows that exist, and masked)
  const int t0 = z * NW + wave, tstep = splits * NW;
  int kidx = 0;
  if (t0 < T) { kidx = key_row(t0); issue_k(kidx); }
  float q[D / 2];
  {
    const int r = row0 + min(c, nrows - 1);                // (rows past the end repeat the last one and are not stored)
    const float* qp = Qh + (size_t)(pq ? pq[r] : r) * D + hb * 4;
#pragma unroll
    for (int i = 0; i < D / 8; ++i) {
      const float4 v = *reinterpret_cast<const float4*>(qp + 8 * i);
      q[4 * i] = v.x; q[4 * i + 1] = v.y; q[4 * i + 2] = v.z; q[4 * i + 3] = v.w;
    }
  }
  f32x16_t o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[db][v] = 0.f;
  // The running maximum starts at a number no score lies below, and that stays one as an exponent of 2: relative to it a
  // score of -inf is a probability of 0 (relative to -inf it would be NaN).
  float m = -3.4028234e38f / fmaxf(1.f, a.scale_log2e), l = 0.f;
  for (int t = t0; t < T; t += tstep) {
    wait_vmcnt<0>();                                       // the K tile has landed
    asm volatile("" ::: "memory");
    float vv[16][DB];
    const int vidx = kidx;
    auto load_v = [&](int j) __attribute__((always_inline)) {      // key 8*(j/4) + 4*hb + j%4: its row number is in that lane
      const int row = __builtin_amdgcn_ds_bpermute(hb * 16 + (8 * (j >> 2) + (j & 3)) * 4, vidx);
      const char* vp = Vh + ((off_t)(uint32_t)row * (D * 4) + (uint32_t)(c * DB * 4));
      if constexpr (DB == 4) {
        const float4 x = *reinterpret_cast<const float4*>(vp);
        vv[j][0] = x.x; vv[j][1] = x.y; vv[j][2] = x.z; vv[j][3] = x.w;
      } else {
        const float2 x = *reinterpret_cast<const float2*>(vp);
        vv[j][0] = x.x; vv[j][1] = x.y;
      }
    };
    // Half of the V rows are requested here, half behind the S products (they are needed last): with all of them in
    // flight the K operands would be left a single register quad, and every fourth product would wait out an LDS read.
#pragma unroll
    for (int j = 0; j < 8; ++j) load_v(j);
    if (t + tstep < T) kidx = key_row(t + tstep);
    __builtin_amdgcn_sched_barrier(0);
    f32x16_t s;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = 0.f;
    // piece 2*i + hb of row c: slot (2*i + hb) ^ (c & 15) below 16 (d=128: pieces 16 .. 31 lie 256 bytes on)
    int ka0 = c * (D * 4) + ((hb ^ (c & 15)) * 16);
    asm volatile("" : "+v"(ka0));
    auto k_piece = [&](int i) __attribute__((always_inline)) {
      return *reinterpret_cast<const float4*>(kt + (ka0 ^ ((i & 7) * 32)) + (i >> 3) * 256);
    };
    constexpr int KA = 4;                                  // K pieces read ahead
    float4 kb[KA];
#pragma unroll
    for (int i = 0; i < KA; ++i) kb[i] = k_piece(i);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < D / 8; ++i) {
      const float4 k4 = kb[i % KA];
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(k4.x, q[4 * i], s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(k4.y, q[4 * i + 1], s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(k4.z, q[4 * i + 2], s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(k4.w, q[4 * i + 3], s, 0, 0, 0);
      if (i + KA < D / 8) kb[i % KA] = k_piece(i + KA);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int j = 8; j < 16; ++j) load_v(j);
    __builtin_amdgcn_sched_barrier(0);
    const int kn = total - t * BN;                         // keys of this tile that exist (>= 1)
    if (kn < BN) {
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (8 * (v >> 2) + 4 * hb + (v & 3) >= kn) s[v] = -INFINITY;
    }
    // m is the running maximum of the raw scores; probabilities are 2^((s - m) scale)
    float tmax = fmaxf(fmaxf(s[0], s[1]), s[2]);
#pragma unroll
    for (int v = 3; v < 15; v += 2) tmax = fmaxf(fmaxf(tmax, s[v]), s[v + 1]);
    tmax = fmaxf(tmax, s[15]);
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
    if (__any(tmax > m)) {
      const float mnew = fmaxf(m, tmax);
      const float alpha = __builtin_amdgcn_exp2f((m - mnew) * a.scale_log2e);
      m = mnew;
      l *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[db][v] *= alpha;
    }
    const float moff = m * a.scale_log2e;
    float lsum[2] = {0.f, 0.f};
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      s[v] = __builtin_amdgcn_exp2f(fmaf(s[v], a.scale_log2e, -moff));
      lsum[v & 1] += s[v];
    }
    l += lsum[0] + lsum[1];                                // (this half-wave's keys; the halves meet at the end)
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      if (j == 8) {
        // All V rows have landed before the next K tile is requested: the compiler does not know of the direct
        // loads, so a wait of its own for a V row would wait for them too.
        wait_vmcnt<0>();
        __builtin_amdgcn_sched_barrier(0);
        if (t + tstep < T) issue_k(kidx);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int db = 0; db < DB; ++db) o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vv[j][db], s[j], o[db], 0, 0, 0);
    }
  }
  __syncthreads();                                         // every wave is done with its K tile: the area changes its use
  // value v of column block db is column i*DB + db, i = 8*(v/4) + 4*hb + v%4, of query c
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    float* out = &sk[(wave * 32 + c) * SROW + (8 * (v >> 2) + 4 * hb + (v & 3)) * DB];
    if constexpr (DB == 4) *reinterpret_cast<float4*>(out) = float4{o[0][v], o[1][v], o[2][v], o[3][v]};
    else *reinterpret_cast<float2*>(out) = float2{o[0][v], o[1][v]};
  }
  l += __shfl_xor(l, 32);
  if (hb == 0) { sm[wave][c] = l > 0.f ? m * a.scale_log2e : -INFINITY; sl[wave][c] = l; }
  __syncthreads();
  // O = sum_w 2^(m_w - M) O_w / sum_w 2^(m_w - M) l_w, 2 NW threads a query; a wave without a tile, or all of whose
  // scores are -inf, has m = -inf and l = 0.  An empty list gives zero, one whose every score is -inf NaN (as 0 / 0).
  constexpr int TPQ = 2 * NW;
  const int r = tid / TPQ, col = (tid % TPQ) * 4;
  if (r >= nrows) return;
  float M = -INFINITY;
#pragma unroll
  for (int w = 0; w < NW; ++w) M = fmaxf(M, sm[w][r]);
  float wt[NW], L = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    wt[w] = M > -INFINITY ? exp2f(sm[w][r] - M) : 0.f;
    L = fmaf(wt[w], sl[w][r], L);
  }
  float inv, *out;
  const size_t pr = ((size_t)h * a.splits + z) * a.N + row0 + r;
  if (splits > 1) {                                        // a partial result: as it is, with its reference and sum
    inv = 1.f;
    out = a.part_o + pr * D;
    if (col == 0) {
      a.part_ml[pr * 2] = M; a.part_ml[pr * 2 + 1] = L;
      if (z == 0)                                          // what the pieces that there are not leave
        for (int u = splits; u < a.splits; ++u) {
          a.part_ml[(pr + (size_t)u * a.N) * 2] = -INFINITY; a.part_ml[(pr + (size_t)u * a.N) * 2 + 1] = 0.f;
        }
    }
  } else {
    if (!(M > -INFINITY) && total > 0) L = NAN;
    inv = L > 0.f ? 1.0f / L : L;
    out = (float*)a.O + ((size_t)h * a.N + (pq ? pq[row0 + r] : row0 + r)) * D;
    if (a.splits > 1 && col == 0) a.part_ml[pr * 2 + 1] = PART_DONE;
  }
#pragma unroll
  for (int cc = 0; cc < D; cc += TPQ * 4) {
    float4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float4 y = *reinterpret_cast<const float4*>(&sk[(w * 32 + r) * SROW + col + cc]);
      x.x = fmaf(wt[w], y.x, x.x); x.y = fmaf(wt[w], y.y, x.y); x.z = fmaf(wt[w], y.z, x.z); x.w = fmaf(wt[w], y.w, x.w);
    }
    *reinterpret_cast<float4*>(out + col + cc) = float4{x.x * inv, x.y * inv, x.z * inv, x.w * inv};
  }
}

// The partial results of a row's up to `splits` workgroups: O = sum_z 2^(M_z - M) O_z / sum_z 2^(M_z - M) L_z.  Their list
// has a key: NaN where no score is above -inf.
template <int D>
__global__ __launch_bounds__(256) void attn_merge_f32(AttnArgs a, int splits) {
  constexpr int LPR = D / 4;
  const int h = blockIdx.y, pos = blockIdx.x * (256 / LPR) + threadIdx.x / LPR, col = (threadIdx.x % LPR) * 4;
  if (pos >= a.N) return;
  float M = -INFINITY, L = 0.f, ms[F32_MAX_SPLITS], ls[F32_MAX_SPLITS];
  float4 os[F32_MAX_SPLITS] = {}, x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int z = 0; z < F32_MAX_SPLITS; ++z) {
    const size_t pr = ((size_t)h * splits + min(z, splits - 1)) * a.N + pos;
    ms[z] = z < splits ? a.part_ml[pr * 2] : -INFINITY;
    ls[z] = a.part_ml[pr * 2 + 1];
  }
  if (ls[0] == PART_DONE) return;
#pragma unroll
  for (int z = 0; z < F32_MAX_SPLITS; ++z)                 // (pieces that there are not have no row)
    if (ms[z] > -INFINITY) os[z] = *reinterpret_cast<const float4*>(a.part_o + (((size_t)h * splits + z) * a.N + pos) * D + col);
#pragma unroll
  for (int z = 0; z < F32_MAX_SPLITS; ++z) M = fmaxf(M, ms[z]);
#pragma unroll
  for (int z = 0; z < F32_MAX_SPLITS; ++z) {
    if (!(ms[z] > -INFINITY)) { if (z < splits) L += ls[z]; continue; }      // 0, or NaN for scores that are
    const float w = exp2f(ms[z] - M);
    L = fmaf(w, ls[z], L);
    x.x = fmaf(w, os[z].x, x.x); x.y = fmaf(w, os[z].y, x.y); x.z = fmaf(w, os[z].z, x.z); x.w = fmaf(w, os[z].w, x.w);
  }
  const float inv = L > 0.f ? 1.0f / L : NAN;
  const int tok = a.perm_q ? a.perm_q[(size_t)h * a.N + pos] : pos;
  *reinterpret_cast<float4*>((float*)a.O + ((size_t)h * a.N + tok) * D + col) = float4{x.x * inv, x.y * inv, x.z * inv, x.w * inv};
}

// ------------------------------------------------------------------------------------------
// merge of the chunks of cut key lists
// ------------------------------------------------------------------------------------------
// O = sum_s 2^((m_s - m) scale) O_s / sum_s 2^((m_s - m) scale) l_s for every row of the cut query tiles,
// with m = max_s m_s.  Every m_s is finite; a chunk all of whose scores are -inf has l_s = 0 and O_s = 0 (under the lowest
// reference there is), and where that is true of every chunk the row is NaN, as 0 / 0.
// MERGE_GROUPS workgroups a head and row group go over the tiles: mostly there is little or nothing to merge, and one for every
// slot, 15 360 for 30 heads, took 5 us to find that out.
constexpr int MERGE_GROUPS = 16;
template <int D>
__global__ __launch_bounds__(256) void attn_merge(AttnArgs a, const int32_t* __restrict__ merge,
                                                  const int32_t* __restrict__ nmerge) {
  // blockIdx.z takes every gridDim.z-th group of rows; the (at most 16) chunks of a row are loaded together,
  // not one after the other: the kernel is a handful of dependent round trips either way, so what counts is
  // how many of its loads are in flight at once.
  constexpr int MAXP = 16;                       // most chunks a list is cut into (plan_tiles)
  const int h = blockIdx.y, n = nmerge[h];
  for (int e = blockIdx.x; e < n; e += gridDim.x) {
    const int32_t* ml = merge + ((size_t)h * a.slots + e) * 4;
    const int row0 = ml[0], nrows = ml[1], slot0 = ml[2], pieces = min(ml[3], MAXP);
    const int32_t* pq = a.perm_q ? a.perm_q + (size_t)h * a.N : nullptr;
    bf16raw* Oh = (bf16raw*)a.O + (size_t)h * a.N * D;
    constexpr int LPR = D / 4;                     // lanes per row, four columns each
    const int col = (threadIdx.x % LPR) * 4;
    for (int r = blockIdx.z * (256 / LPR) + threadIdx.x / LPR; r < nrows; r += gridDim.z * (256 / LPR)) {
      float ms[MAXP], ls[MAXP];
      float4 os[MAXP];
#pragma unroll
      for (int s = 0; s < MAXP; ++s) {
        const size_t so = ((size_t)h * a.slots + slot0 + min(s, pieces - 1)) * a.BM + r;
        ms[s] = a.part_ml[so * 2];
        ls[s] = a.part_ml[so * 2 + 1];
        os[s] = *reinterpret_cast<const float4*>(a.part_o + so * D + col);
      }
      float m = -INFINITY;
#pragma unroll
      for (int s = 0; s < MAXP; ++s) if (s < pieces) m = fmaxf(m, ms[s]);
      float l = 0.f;
      float4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < MAXP; ++s) {
        if (s < pieces) {                          // in chunk order, as before: the sums are the same to the bit
          const float w = __builtin_amdgcn_exp2f((ms[s] - m) * a.scale_log2e);
          l = fmaf(w, ls[s], l);
          o.x = fmaf(w, os[s].x, o.x); o.y = fmaf(w, os[s].y, o.y); o.z = fmaf(w, os[s].z, o.z); o.w = fmaf(w, os[s].w, o.w);
        }
      }
      const float inv = l > 0.f ? 1.0f / l : NAN;
      const int tok = pq ? pq[row0 + r] : row0 + r;
      uint2 out;
      out.x = pack_bf16x2(o.x * inv, o.y * inv);
      out.y = pack_bf16x2(o.z * inv, o.w * inv);
      *reinterpret_cast<uint2*>(Oh + (size_t)tok * D + col) = out;
    }
  }
}

// ------------------------------------------------------------------------------------------
// tile shapes of the bf16 kernel: waves per workgroup NW (32 queries each), pipeline stages NBUF, and MINB = the
// waves per SIMD the register budget is set for (the second __launch_bounds__ argument)
#ifndef A64_NW
#define A64_NW 8
#endif
#ifndef A64_NBUF
#define A64_NBUF 4
#endif
#ifndef A64_MINB
#define A64_MINB 4
#endif
#ifndef A128_NW
#define A128_NW 8
#endif
#ifndef A128_NBUF
#define A128_NBUF 4
#endif
#ifndef A128_MINB
#define A128_MINB 2
#endif
// 32-column blocks of V whose operands are requested before the soft-max arithmetic (the rest follow it)
#ifndef A64_VPRE
#define A64_VPRE 0
#endif
#ifndef A128_VPRE
#define A128_VPRE 2
#endif

// Queries per workgroup.  The bf16 kernel comes in two shapes: eight waves (256 queries, a ring of four stages),
// and four waves (128 queries, two stages, twice the workgroups per CU) for query clusters too small to fill
// the first without long tails (a cluster of 273 queries is 256 + 17 in one shape, 128 + 128 + 17 in the other).
static bool attn_small_shape(int N, int Cq) { return Cq > 1 && N / Cq < 768; }
int attn_block_rows(int dtype, int d, int N, int Cq) {
  if (dtype != ADACLUSTER_BF16) return 32;
  if (attn_small_shape(N, Cq)) return 128;
  return d == 64 ? A64_NW * 32 : A128_NW * 32;
}
// Shape of a dense launch: queries a workgroup, and pieces of the key list (unnormalised partial results and a merge, as for cut
// lists).  A launch of few query tiles leaves most of the chip idle with 256 queries a workgroup, so it takes 128 and, while that
// fills less than a round, pieces.  Priced in steps of a key tile (0.9 us at d=64, 1.6 at d=128) by the workgroups on a CU, heads
// dealt to the XCDs whole and those left over in eighths: they share its matrix cores.  At d=64 a workgroup alone is slower than its
// share, and what counts for 128 queries is the mean CU; at d=128 three of 128, of which two fit at once, take less than two of 256,
// more again by the mean.  A workgroup costs a few steps besides its own; a merge its launch and 4 to 8 TB/s on its partial results.
// The figures are fitted to the times of 261 launches of 500-33 000 rows, 168 of them in every form (profiles/dense_shapes.txt has
// some on both sides of every choice): the chosen form takes 1.004 (d=64) and 1.008 (d=128) of the best one's time in the geometric
// mean.  (In the table 9 x 14 399, d=64, 557 and 579, and 5 x 27 679, d=128, 1 998 and 2 120, are the worst.)
// The shape, and with it the rounding of a row, depends on the number of heads.
DenseShape attn_dense_shape(int dtype, int d, int H, int N) {
  if (dtype != ADACLUSTER_BF16) return {32, 1};
  const bool w64 = d == 64;
  const int T = (N + 63) / 64, nq = (N + 127) / 128;
  auto load = [&](long long tiles) { return (double)(H / 8 * tiles + H % 8 * ((tiles + 7) / 8)) / 32.0; };      // workgroups a CU, in the busiest XCD
  const double wide = load((N + 255) / 256), kw = w64 && wide > 0.97 ? fmax(2.0, ceil(wide)) : ceil(wide);      // (d=64, one for every CU: some get two)
  double best = w64 ? (kw > 1.0 ? 0.92 * kw : 0.93 + 0.24 * wide) * (T + 8) : (kw > 1.0 ? 0.93 * kw : 0.8) * (T + 2);
  DenseShape r{256, 1};
  for (int want = 1; want <= 16 && (want == 1 || nq * want <= SPLIT_SLOTS); ++want) {
    const int per = (T + want - 1) / want, pieces = (T + per - 1) / per;
    if (pieces != want || (want > 1 && per < 2)) continue;      // (no empty piece)
    const double x = load((long long)nq * pieces), k = ceil(x);
    const double share = !w64 ? (k > 3.0 ? 0.73 * x : k > 1.0 ? 0.6 * k : 0.7) : pieces > 1 ? fmax(0.8, 0.6 * x) : fmax(0.72, 0.28 + 0.52 * x);
    const double partial = (double)H * N * pieces * (d + 2) * 1e-6;
    const double merge = pieces == 1 ? 0.0 : w64 ? 14.0 + partial / 0.9 : 6.0 + 2.0 * partial / 1.6;
    const double cost = share * (per + (w64 && pieces > 1 ? 4 : 2)) + merge;
    if (cost < best) { best = cost; r = {128, pieces}; }
  }
  return r;
}
int attn_block_rows_min(int dtype) { return dtype == ADACLUSTER_BF16 ? 128 : 32; }
int attn_block_rows_max(int dtype) { return dtype == ADACLUSTER_BF16 ? 256 : 32; }

// The launch of a kernel that takes its tiles by pick_tile: `most` bounds the tiles of a head.
static dim3 pick_tile_grid(int H, int most, int splits, int resident) {
  const unsigned x = (most + 7) / 8 * 8;
  return H > PICK_HEADS ? dim3(x, H) : splits > 1 ? dim3(H * x + min((splits - 1) * H * x, 8 * 3 * resident)) : dim3(H * x);
}

size_t attn_krow_stride(int N) { return (size_t)(N + 63) / 64 * 64 + KROW_PAD; }

// Whether the planning step writes the key rows of every list to a table, [H][Cq][N + padding] integers.  The fp32 kernel can
// also search them in the ranges, tile by tile: 6-7 % slower with tens of clusters (one head of 4 096, d=64, 32 clusters
// 69 and 76 us for the call; three of 5 007, d=128, 65 clusters 251 and 266), 15-34 % with hundreds and thousands (4 x 12 000,
// d=64, 1 024 clusters 1 365 and 1 832; 24 x 20 000, d=128, 512 clusters 6.5 and 7.5 ms).  So the table stays, unless it takes
// more than 1 GiB and more than copies of K and V would (24 x 180 000 rows with 4 096 clusters: 71 GB; all else in the
// workspace 11): a call has to fit the card.  Heads of 4 GiB and more need 64-bit offsets, which only the searching form has.
bool attn_rows_listed(int dtype, int d, int H, int N, int Cq) {
  if (dtype == ADACLUSTER_BF16) return true;
  const bool large = Cq > 2 * d && (size_t)H * Cq * attn_krow_stride(N) * 4 > ((size_t)1 << 30);
  return !large && (size_t)N * d * 4 < ((size_t)1 << 32);
}

int attn_tile_record() { return TILE_REC; }
int attn_split_slots() { return SPLIT_SLOTS; }
// Tiles of a head that the grid of a sparse launch is sized for, at least what it can have.  Workgroups go to the CUs in turn, so
// those without work leave places empty that a small launch would have used: where no list is cut, none for pieces.
static bool lists_may_be_cut(int N) { return (N + 63) / 64 > 2 * MIN_CHUNK; }
int attn_most_tiles(int dtype, int N, int Cq, int BM, int maxtiles) {
  return dtype == ADACLUSTER_F32 || !lists_may_be_cut(N) ? N / BM + Cq + 1 : maxtiles;      // (an fp32 list has no records for its pieces)
}
static int attn_resident(int d, int BM) { return 256 * (BM == 128 ? 2 : 1) * (d == 64 ? 2 : 1); }      // workgroups of the bf16 kernel
int attn_deal_segs(int dtype, int d, int H, int N, int Cq, bool top_p) {
  const int BM = attn_block_rows(dtype, d, N, Cq);
  return dtype == ADACLUSTER_F32 ? deal_segs_f32(d, H, N, Cq, top_p) : deal_segs_bf16(BM, attn_resident(d, BM), H, N, Cq);
}
static int deal_entries(int dtype, int d, int H, int N, int Cq, int segs, int most) {
  return dtype == ADACLUSTER_F32 ? deal_entries_f32(d, H, N, Cq, segs, most) : deal_list(H, segs, most);
}
size_t attn_deal_ints(int dtype, int d, int H, int N, int Cq, int segs, int most) {
  return segs ? DEAL_PARTS + 8 * (size_t)(DEAL_HEAD + deal_entries(dtype, d, H, N, Cq, segs, most)) : 0;
}

int attn_f32_splits(int H, int N, int Cq) { return f32_splits(H, N, Cq); }

// The rule: the number that ends first, the smallest of equals.  A piece takes a wave's share of the list's key tiles (as many
// as a list can have) and half a tile for its start and end; the workgroups that share a CU take turns, so a round lasts as
// long as it has workgroups a CU (alone on one, a little longer), and one that is not full a quarter of the way to a full one
// longer, unless it is the first: not every CU gets its share of those.
// us of a dense call with 1, 2, 3 and 4 pieces (chosen: the one in brackets): d=128, 3 x 2 088, 27 tiles an XCD: 87 [86] 108 94;
// 1 x 2 101 (9): 86 53 [41] 53; 4 x 3 076 (52): 215 224 [198] 209; 12 x 467 (24): [30] 35 38 40; d=64, 1 x 4 746 (19): 100 95 [71]
// 76; 12 x 772 (48): 41 [37] 43 42; 8 x 2 414 (80): 134 123 131 [128].  (1.6 pieces a place, whatever they leave of a round, took
// 108, 53, 224, 40, 76, 43 and 122 us; four for every list where those are fewer than 1 024, 92, 51, 194, 39, 75, 40 and 124.)
// (The turns are a table: 380 of them by division were 5 us of a call.)
template <int D>
struct PieceTurns {
  static constexpr int RESIDENT = f32_resident(D), FULL = RESIDENT / 32;      // FULL: workgroups of a CU
  int of[RESIDENT][F32_MAX_SPLITS];                                           // in 32nds of one alone on every CU
  constexpr PieceTurns() : of{} {
    for (int rest = 1; rest < RESIDENT; ++rest)
      for (int sp = 1; sp <= F32_MAX_SPLITS; ++sp) {
        const int n = rest * sp, f = n / RESIDENT, r = n % RESIDENT, k = (r + 31) / 32;
        of[rest][sp - 1] = 32 * FULL * f + (r == 0 ? 0 : f > 0 ? 24 * k + 8 * FULL : k > 1 ? 32 * k : 33);
      }
  }
};
template <int D>
static Pieces f32_pieces(int N) {
  static constexpr PieceTurns<D> turns{};
  static_assert(F32_MAX_SPLITS <= 4 && PieceTurns<D>::RESIDENT <= 96, "Pieces holds them");
  const int keys = (N + 31) / 32;
  long long len[F32_MAX_SPLITS];
  for (int i = 0; i < F32_MAX_SPLITS; ++i) len[i] = 2ll * ((keys + (i + 1) * F32_WAVES - 1) / ((i + 1) * F32_WAVES)) + 1;
  Pieces p{};
  for (int rest = 1; rest < PieceTurns<D>::RESIDENT; ++rest) {
    long long best = turns.of[rest][0] * len[0];
    int more = 0;
    for (int i = 1; i < F32_MAX_SPLITS; ++i) {
      const long long t = turns.of[rest][i] * len[i];
      if (t < best) { best = t; more = i; }
    }
    p.of[rest / 32] |= (uint64_t)more << (2 * (rest % 32));
  }
  return p;
}

static Deal deal_of(int dtype, int d, int H, int N, int Cq, int segs, int most, int32_t* deal, int32_t* planned) {
  Deal dl{};
  if (!segs) return dl;
  dl.parts = deal; dl.lists = deal + DEAL_PARTS; dl.planned = planned; dl.cap = deal_entries(dtype, d, H, N, Cq, segs, most); dl.segs = segs; dl.H = H;
  if (dtype == ADACLUSTER_F32 && attn_f32_splits(H, N, Cq) > 1) {
    dl.f32_round = f32_resident(d);
    dl.pieces = d == 64 ? f32_pieces<64>(N) : f32_pieces<128>(N);
  }
  return dl;
}
bool plan_reads_lengths(int Cq) { return Cq <= PLAN_BESIDE; }
int launch_plan_sparse(hipStream_t s, int dtype, int d, int H, int Cq, int cap, int maxr, int maxtiles, int BM,
                       const int32_t* q_offs, int q_offs_stride, const int32_t* k_offs, int k_offs_stride,
                       const int32_t* k_count, const int32_t* sel_idx, const int32_t* sel_cnt,
                       int32_t* rng_start, int32_t* rng_pre, int32_t* rng_cnt, int32_t* tiles, int32_t* ntiles,
                       int32_t* merge, int32_t* nmerge, int row_scale, int32_t* krow, size_t kstride,
                       const int32_t* perm_k, int N, const int32_t* lengths, int segs, int most, int32_t* deal, int32_t* planned) {
  const int split = dtype == ADACLUSTER_BF16 ? 1 : 0;
  const TilePlan tp{lengths, q_offs, q_offs_stride, maxtiles, BM, SPLIT_SLOTS, split, tiles, ntiles, merge, nmerge, deal_of(dtype, d, H, N, Cq, segs, most, deal, planned)};
  if (lengths && plan_reads_lengths(Cq)) {
    const auto plan = segs ? plan_sparse<true, true> : plan_sparse<true, false>;
    plan<<<dim3(H, Cq + 1), 256, plan_ints(Cq, segs != 0) * 4, s>>>(
        Cq, cap, maxr, row_scale, k_offs, k_offs_stride, k_count, sel_idx, sel_cnt, rng_start, rng_pre, rng_cnt, krow, kstride, perm_k, N, tp);
  } else {
    plan_sparse<false, false><<<dim3(H, Cq), 256, 0, s>>>(Cq, cap, maxr, row_scale, k_offs, k_offs_stride, k_count, sel_idx, sel_cnt, rng_start, rng_pre,
                                                          rng_cnt, krow, kstride, perm_k, N, tp);
    const auto plan = segs ? plan_tiles<true> : plan_tiles<false>;
    plan<<<H, 256, 0, s>>>(Cq, maxr, maxtiles, BM, SPLIT_SLOTS, split, tp.deal, q_offs, q_offs_stride, rng_pre, rng_cnt, tiles, ntiles, merge, nmerge);
  }
  return hipGetLastError() == hipSuccess ? 0 : ADACLUSTER_E_INTERNAL;
}

int launch_plan_dense(hipStream_t s, int H, int N, int maxtiles, DenseShape shape, int32_t* rng_start, int32_t* rng_pre,
                      int32_t* rng_cnt, int32_t* tiles, int32_t* ntiles, int32_t* merge, int32_t* nmerge, int row_scale, int32_t* krow, size_t kstride) {
  plan_dense<<<dim3(H, 9), 256, 0, s>>>(N, maxtiles, shape.BM, shape.pieces, SPLIT_SLOTS, row_scale, rng_start, rng_pre, rng_cnt, tiles, ntiles, merge,
                                        nmerge, krow, kstride);
  return hipGetLastError() == hipSuccess ? 0 : ADACLUSTER_E_INTERNAL;
}

int launch_attention(hipStream_t s, int dtype, int d, int H, int N, int Cq, int BM, int most, int maxtiles, float scale,
                     const void* Q, const void* K, const void* V, void* O, const int32_t* perm_q,
                     const int32_t* tiles, const int32_t* ntiles, float* part_o, float* part_ml,
                     const int32_t* merge, const int32_t* nmerge, const int32_t* krow, size_t kstride,
                     const int32_t* rng_start, const int32_t* rng_pre, const int32_t* rng_cnt, int maxr, const int32_t* perm_k,
                     int segs, int32_t* deal) {
  AttnArgs a{Q, K, V, O, perm_q, tiles, ntiles, H, N, Cq, maxtiles,
             scale * 1.4426950408889634f,
             (Cq == 1 || (size_t)4 * N * d <= ((size_t)8 << 20)) ? 1 : 0,
             part_o, part_ml, SPLIT_SLOTS, BM, krow, kstride,
             rng_start, rng_pre, rng_cnt, maxr, perm_k, dtype == ADACLUSTER_F32 ? attn_f32_splits(H, N, Cq) : 1, {}, nullptr, 0};
  const int entries = segs ? deal_entries(dtype, d, H, N, Cq, segs, most) : 0;
  if (segs) { a.deal = deal + DEAL_PARTS; a.deal_stride = DEAL_HEAD + entries; }
  else if (a.splits > 1) a.pieces = d == 64 ? f32_pieces<64>(N) : f32_pieces<128>(N);
  const bool cut = Cq == 1 || lists_may_be_cut(N);
  const dim3 g = segs ? dim3(8 * entries) : dim3((most + 7) / 8 * 8, H);
  if (dtype == ADACLUSTER_BF16) {
    if (BM == 128) {
      if (d == 64) attn_mfma<64, 4, 2, 4, 0><<<g, 256, 0, s>>>(a);
      else attn_mfma<128, 4, 2, 2, 2><<<g, 256, 0, s>>>(a);
    } else {
      if (d == 64) attn_mfma<64, A64_NW, A64_NBUF, A64_MINB, A64_VPRE><<<g, A64_NW * 64, 0, s>>>(a);
      else attn_mfma<128, A128_NW, A128_NBUF, A128_MINB, A128_VPRE><<<g, A128_NW * 64, 0, s>>>(a);
    }
    if (merge && cut) {      // the chunks of cut key lists
      const dim3 gm(MERGE_GROUPS, H, 4);
      if (d == 64) attn_merge<64><<<gm, 256, 0, s>>>(a, merge, nmerge);
      else attn_merge<128><<<gm, 256, 0, s>>>(a, merge, nmerge);
    }
  } else {
    const int splits = a.splits;
    const dim3 g2 = segs ? g : pick_tile_grid(H, min(N, N / 32 + Cq + 1), splits, f32_resident(d)), gm((N + 1024 / d - 1) / (1024 / d), H);
    if (d == 64) { if (krow) attn_f32<64, true><<<g2, F32_WAVES * 64, 0, s>>>(a); else attn_f32<64, false><<<g2, F32_WAVES * 64, 0, s>>>(a); }
    else { if (krow) attn_f32<128, true><<<g2, F32_WAVES * 64, 0, s>>>(a); else attn_f32<128, false><<<g2, F32_WAVES * 64, 0, s>>>(a); }
    if (splits > 1) {
      if (d == 64) attn_merge_f32<64><<<gm, 256, 0, s>>>(a, splits);
      else attn_merge_f32<128><<<gm, 256, 0, s>>>(a, splits);
    }
  }
  return hipGetLastError() == hipSuccess ? 0 : ADACLUSTER_E_INTERNAL;
}

}  // namespace adac
