// Critical-cluster selection: centroid scores (Eq. 1 / Eq. 2, Algorithm 2), arg-top-k (Alg. 3
// line 8) and the top-p budget.
//
// The score matrix is tiny (Cq x Ck x d per head), so it is evaluated in fp64, term by term in ascending
// dimension order, with the bits a rounded multiply followed by a rounded add would give (score_kernel says
// why its fused multiply-adds do).  That makes every bit of a score, and therefore every selected index set,
// reproducible by a CPU implementation.  Floating-point contraction by the compiler is switched off for this
// file for the same reason.
#include "common.h"
#include "launch.h"

#include <atomic>
#include <type_traits>

#pragma clang fp contract(off)

namespace adac {

struct SelectCfg {
  int Cq, cap, d, lds_cap;
  int score_mode, select_mode, topk;
  double top_p, scale;
};

// exp(x), x <= 0, from rounded +,* only: k = rint(x log2 e); r = (x - k ln2_hi) - k ln2_lo;
// degree-13 Taylor polynomial in Horner form; scaled by 2^k.  0 below -700.
__device__ double exp_det(double x) {
#pragma clang fp contract(off)
  if (x < -700.0) return 0.0;
  const double k = rint(x * 1.4426950408889634);
  const double r = (x - k * 0.693147180369123816490) - k * 1.90821492927058770002e-10;
  // 1/n!, each the correctly rounded quotient of 1 and the (exact) double n!; folded at compile time,
  // which rounds as the device would
  constexpr double c[14] = {1.0 / 1.0, 1.0 / 1.0, 1.0 / 2.0, 1.0 / 6.0, 1.0 / 24.0, 1.0 / 120.0, 1.0 / 720.0,
                            1.0 / 5040.0, 1.0 / 40320.0, 1.0 / 362880.0, 1.0 / 3628800.0, 1.0 / 39916800.0,
                            1.0 / 479001600.0, 1.0 / 6227020800.0};
  double p = c[13];
#pragma unroll
  for (int n = 12; n >= 0; --n) p = p * r + c[n];
  return ldexp(p, (int)k);
}

// monotone map double -> uint64 (larger double = larger key); -inf is the smallest key
__device__ __forceinline__ uint64_t order_key(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// Scores of every (query cluster, key cluster) pair: S[h][i][j], -inf for an empty key cluster, 0 for a head
// that attends to everything.  A thread owns a key cluster and reads its row ONCE for QG query clusters, whose
// centroids wait in LDS split by sign:
//   (q, 0) where q's sign bit is clear, (0, q) where it is set.
// Every score is the pair of chains  sp += q+ * k+,  sn += q- * k-  in ascending dimension order with
// k+/k- = max(c,0)/min(c,0) (Algorithm 2), box max/min (Eq. 1), or c itself with q- = 0 (plain dot product).
// The term of the sign q does not have is an exact zero, which leaves its chain as it was, so each chain sees
// exactly the terms it owns.  q and k are float values, so a product is exact in double (48 significant bits
// at most, exponents far inside the range) and the fused multiply-add rounds once, exactly where the add of a
// separately rounded product would: the same bits as multiply-then-add at twice the rate.
// (One workgroup per query cluster reading every key row itself was bound by L2 traffic: 65 reads of a head's centroid table.)
// What bounds it: large tables the LDS pipe (a 16-byte broadcast read per two fused multiply-adds; two rows a thread
// halve the reads and cost as much in waves), small ones the trips to the rows, which finalize_centroids has just written
// on other XCDs.  So eight pieces of a row are in flight a step, the first of them from the kernel's first instructions on
// (four, behind the counts, sizes and flags before): 5 heads x 110 clusters, d=128, 17 -> 10 us (boxes 22 -> 10),
// 12 x 330, d=128, 24 -> 18 (33 -> 20), 24 x 1171, d=128, 92 -> 69 (129 -> 73), 30 x 600, d=64, 33 -> 30 (42 -> 31).
// The query values as scalar operands (scalar loads from a table prepared by another kernel, no LDS) took more than
// twice as long: the scalar cache delivers far less than the LDS.
constexpr int SCORE_THREADS = 128;

template <int QG, int D, bool BOX>
__global__ __launch_bounds__(SCORE_THREADS) void score_kernel(SelectCfg cfg, const float* __restrict__ q_cent,
                                                              const float* __restrict__ k_cent,
                                                              const float* __restrict__ k_bmin,
                                                              const float* __restrict__ k_bmax,
                                                              const int32_t* __restrict__ k_sizes,
                                                              const int32_t* __restrict__ k_count,
                                                              const int32_t* __restrict__ full_flag,
                                                              double* __restrict__ S) {
  constexpr int B4 = 8, STEPS = D / (4 * B4);      // 16-byte pieces of a row per step
  __shared__ __attribute__((aligned(16))) double2 qs[QG * D];
  const int h = blockIdx.z, i0 = blockIdx.y * QG, tid = threadIdx.x;
  const int j = blockIdx.x * SCORE_THREADS + tid;
  // (rows past the count exist: the tables hold `cap` of them)
  const size_t row = ((size_t)h * cfg.cap + min(j, cfg.cap - 1)) * D;
  const float4* rpos = reinterpret_cast<const float4*>((BOX ? k_bmax : k_cent) + row);
  const float4* rneg = reinterpret_cast<const float4*>((BOX ? k_bmin : k_cent) + row);
  float4 pb[B4], nb[B4];
#pragma unroll
  for (int u = 0; u < B4; ++u) { pb[u] = rpos[u]; if (BOX) nb[u] = rneg[u]; }
  const int kc = min(k_count[h], cfg.lds_cap);
  if ((int)blockIdx.x * SCORE_THREADS >= kc) return;
  const bool dot = cfg.score_mode == ADACLUSTER_SCORE_DOT, all = full_flag[h] != 0;
  for (int e = tid; e < QG * D; e += SCORE_THREADS) {
    const int i = min(i0 + e / D, cfg.Cq - 1);     // (the last group repeats the last cluster; not stored)
    const float q = q_cent[((size_t)h * cfg.Cq + i) * D + e % D];
    const bool neg = (__float_as_uint(q) >> 31) != 0u;
    double2 v;
    v.x = (dot || !neg) ? (double)q : 0.0;
    v.y = (!dot && neg) ? (double)q : 0.0;
    qs[e] = v;
  }
  __syncthreads();
  if (j >= kc) return;          // (a wave without a cluster reads no LDS: 30 x 1 063 lists of some 50 clusters, d=64, 76 -> 53 us)
  double sp[QG], sn[QG];
#pragma unroll
  for (int g = 0; g < QG; ++g) { sp[g] = 0.0; sn[g] = 0.0; }
  if (!all) {
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
      float4 pc[B4], nc[B4];
#pragma unroll
      for (int u = 0; u < B4; ++u) {
        pc[u] = pb[u]; if (BOX) nc[u] = nb[u];
        if (st + 1 < STEPS) { pb[u] = rpos[(st + 1) * B4 + u]; if (BOX) nb[u] = rneg[(st + 1) * B4 + u]; }
      }
#pragma unroll
      for (int u4 = 0; u4 < B4; ++u4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int t = (st * B4 + u4) * 4 + u;
          const float pv = u == 0 ? pc[u4].x : u == 1 ? pc[u4].y : u == 2 ? pc[u4].z : pc[u4].w;
          const float nv = !BOX ? pv : u == 0 ? nc[u4].x : u == 1 ? nc[u4].y : u == 2 ? nc[u4].z : nc[u4].w;
          const double kp = (double)((BOX || dot) ? pv : fmaxf(pv, 0.f));
          const double kn = (double)((BOX || dot) ? nv : fminf(nv, 0.f));
#pragma unroll
          for (int g = 0; g < QG; ++g) {
            const double2 q2 = qs[g * D + t];
            sp[g] = __fma_rn(q2.x, kp, sp[g]);
            sn[g] = __fma_rn(q2.y, kn, sn[g]);
          }
        }
      }
    }
  }
  const int nj = k_sizes[(size_t)h * cfg.cap + j];
  double* out = S + ((size_t)h * cfg.Cq + i0) * cfg.cap + j;
#pragma unroll
  for (int g = 0; g < QG; ++g)
    if (i0 + g < cfg.Cq) out[(size_t)g * cfg.cap] = nj == 0 ? -INFINITY : all ? 0.0 : sp[g] + sn[g];
}

// One block per (query cluster, head).  Dynamic LDS: key[cap] (uint64) + flag[cap] (int).
// Top-p, top-k and the keys of the lists (sel_keys) are compiled apart: in one kernel, whose registers and steps a top-k
// without them then has too, top-k over 30 x 65 lists of 50 clusters took 9.4 us, now 8.1, over 48 x 1 000 140 and 115.
// D > 0: small tables are scored here, a key cluster a thread, by the chains of score_kernel: the launch before took 7 us and a
// trip to the scores, this 2 (a workgroup reads its head's whole table: see the line in launch_select).
struct ScoreTables { const float* q_cent; const float* k_cent; const float* k_bmin; const float* k_bmax; };
template <bool TOPP, bool KEYS, int D, bool BOX>
__global__ __launch_bounds__(256) void select_kernel(SelectCfg cfg, const double* __restrict__ S, ScoreTables t,
                                                     const float* __restrict__ q_mean_norm,
                                                     const int32_t* __restrict__ k_sizes,
                                                     const int32_t* __restrict__ k_count,
                                                     const int32_t* __restrict__ full_flag,
                                                     int32_t* __restrict__ sel_idx, int32_t* __restrict__ sel_cnt,
                                                     int32_t* __restrict__ sel_keys) {
#pragma clang fp contract(off)
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  double* sval = reinterpret_cast<double*>(smem);                        // [cap] score, then weight
  uint64_t* skey = reinterpret_cast<uint64_t*>(smem + (size_t)cfg.lds_cap * 8);   // [lds_cap]
  int32_t* sflag = reinterpret_cast<int32_t*>(smem + (size_t)cfg.lds_cap * 16);   // [lds_cap]
  __shared__ int32_t wsum[4], wsum2[4];
  __shared__ int32_t s_take, s_digit, s_krem, s_all;
  __shared__ int32_t hist[256], dup[256];
  __shared__ double s_max;
  __shared__ double swmax[4];

  const int h = blockIdx.y, i = blockIdx.x, tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  bool use_thr = false;          // top-k by threshold key: selected = key > thr_key, or == thr_key among the first thr_rem
  uint64_t thr_key = 0;
  int thr_rem = 0;
  constexpr int B4 = 8, STEPS = D / (4 * B4);      // as in score_kernel
  float4 pb[B4], nb[B4];
  const float4 *rpos = nullptr, *rneg = nullptr;
  if constexpr (D > 0) {
    const size_t row = ((size_t)h * cfg.cap + min(tid, cfg.cap - 1)) * D;
    rpos = reinterpret_cast<const float4*>((BOX ? t.k_bmax : t.k_cent) + row);
    rneg = reinterpret_cast<const float4*>((BOX ? t.k_bmin : t.k_cent) + row);
#pragma unroll
    for (int u = 0; u < B4; ++u) { pb[u] = rpos[u]; if (BOX) nb[u] = rneg[u]; }
  }
  const int kc = min(k_count[h], cfg.lds_cap);
  const bool all = full_flag[h] != 0;
  // ---- scores of this query cluster
  if constexpr (D > 0) {
    __shared__ __attribute__((aligned(16))) double2 qs[D];
    const bool dot = cfg.score_mode == ADACLUSTER_SCORE_DOT;
    if (tid < D) {
      const float q = t.q_cent[((size_t)h * cfg.Cq + i) * D + tid];
      const bool neg = (__float_as_uint(q) >> 31) != 0u;
      qs[tid] = double2{(dot || !neg) ? (double)q : 0.0, (!dot && neg) ? (double)q : 0.0};
    }
    const int nj = k_sizes[(size_t)h * cfg.cap + min(tid, cfg.cap - 1)];
    __syncthreads();
    if (tid < kc) {                                // (kc <= 256)
      double sp = 0.0, sn = 0.0;
#pragma unroll
      for (int st = 0; st < STEPS; ++st) {
        float4 pc[B4], nc[B4];
#pragma unroll
        for (int u = 0; u < B4; ++u) {
          pc[u] = pb[u]; if (BOX) nc[u] = nb[u];
          if (st + 1 < STEPS) { pb[u] = rpos[(st + 1) * B4 + u]; if (BOX) nb[u] = rneg[(st + 1) * B4 + u]; }
        }
#pragma unroll
        for (int u4 = 0; u4 < B4; ++u4) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float pv = u == 0 ? pc[u4].x : u == 1 ? pc[u4].y : u == 2 ? pc[u4].z : pc[u4].w;
            const float nv = !BOX ? pv : u == 0 ? nc[u4].x : u == 1 ? nc[u4].y : u == 2 ? nc[u4].z : nc[u4].w;
            const double kp = (double)((BOX || dot) ? pv : fmaxf(pv, 0.f));
            const double kn = (double)((BOX || dot) ? nv : fminf(nv, 0.f));
            const double2 q2 = qs[(st * B4 + u4) * 4 + u];
            sp = __fma_rn(q2.x, kp, sp);
            sn = __fma_rn(q2.y, kn, sn);
          }
        }
      }
      sval[tid] = nj == 0 ? -INFINITY : all ? 0.0 : sp + sn;
    }
  } else {
    const double* sr = S + ((size_t)h * cfg.Cq + i) * cfg.cap;
    for (int j = tid; j < kc; j += 256) sval[j] = sr[j];
  }
  __syncthreads();

  if (all || (TOPP && cfg.top_p >= 1.0)) {
    for (int j = tid; j < kc; j += 256) sflag[j] = sval[j] > -INFINITY;
  } else if constexpr (!TOPP) {
    // The topk largest by (score desc, index asc).  No ranks are needed, only the key of the
    // topk-th largest: an MSB-first radix select over the 64-bit order keys (eight 8-bit digits, a
    // 256-bin histogram per digit).  Equal keys at the threshold are resolved by index in the
    // compaction below, which walks the clusters in ascending order anyway.
    int nv = 0;
    for (int j = tid; j < kc; j += 256) {
      const double v = sval[j];
      skey[j] = order_key(v);
      nv += v > -INFINITY;
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) nv += __shfl_xor(nv, o);
    if (lane == 0) wsum[wave] = nv;
    __syncthreads();
    const int nvalid = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    __syncthreads();
    if (nvalid <= cfg.topk) {
      for (int j = tid; j < kc; j += 256) sflag[j] = sval[j] > -INFINITY;
    } else {
      use_thr = true;
      uint64_t prefix = 0;
      int krem = cfg.topk;
      for (int pass = 0; pass < 8; ++pass) {
        const int shift = 56 - 8 * pass;
        hist[tid] = 0;
        __syncthreads();
        for (int j = tid; j < kc; j += 256) {
          const uint64_t k = skey[j];
          if (pass == 0 || (k >> (shift + 8)) == (prefix >> (shift + 8))) atomicAdd(&hist[(int)((k >> shift) & 255)], 1);
        }
        __syncthreads();
        // thread t owns bin 255 - t: an inclusive scan over t counts the keys in higher or equal bins
        const int bin = 255 - tid;
        const int cnt = hist[bin];
        int incl = cnt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) { const int u = __shfl_up(incl, o); if (lane >= o) incl += u; }
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        for (int w = 0; w < wave; ++w) incl += wsum[w];
        const int excl = incl - cnt;
        if (excl < krem && krem <= incl) { s_digit = bin; s_krem = krem - excl; s_all = (krem == incl); }
        __syncthreads();
        prefix |= (uint64_t)s_digit << shift;
        krem = s_krem;
        // every key of the chosen bin is wanted: the threshold is the bin's lower edge, no ties to split
        if (s_all && prefix != 0) { prefix -= 1; krem = 0; break; }
      }
      thr_key = prefix; thr_rem = krem;
    }
  } else {
    // weights w_j = n_j exp(alpha (S_j - max S)); order by (w desc, j asc); shortest prefix
    // whose running sum reaches top_p * total
    {
      // the maximum does not depend on the order it is taken in
      double m = -INFINITY;
      for (int j = tid; j < kc; j += 256) m = fmax(m, sval[j]);
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) m = fmax(m, __shfl_xor(m, o));
      if (lane == 0) swmax[wave] = m;
      __syncthreads();
      if (tid == 0) s_max = fmax(fmax(swmax[0], swmax[1]), fmax(swmax[2], swmax[3]));
      __syncthreads();
    }
    const double alpha = (double)q_mean_norm[(size_t)h * cfg.Cq + i] * cfg.scale;
    const double mx = s_max;
    for (int j = tid; j < kc; j += 256) {
      const int nj = k_sizes[(size_t)h * cfg.cap + j];
      double w = 0.0;
      if (nj > 0) w = (double)nj * exp_det(alpha * (sval[j] - mx));
      const bool valid = sval[j] > -INFINITY;
      sval[j] = w;
      // invalid (empty) clusters sort after everything else
      skey[j] = valid ? order_key(w) : 0ull;
      sflag[j] = valid;
    }
    __syncthreads();
    if (kc <= 64) {
      // A wave does the rest without a barrier: whole keys for the ranks, and both sums in every lane.  (As below, 48 x 1 000
      // lists of 8 clusters take 137 us, so 82; of 64 219 and 182; 30 x 65 lists of 50 12.6 and 11.6.)
      if (wave == 0) {
        const bool valid = lane < kc && sflag[lane] != 0;
        const double w = lane < kc ? sval[lane] : 0.0;
        const uint64_t k1 = lane < kc ? skey[lane] : 0ull;
        int r = 0;
#pragma unroll 8
        for (int t = 0; t < kc; ++t) { const uint64_t kt = skey[t]; r += (kt > k1) || (kt == k1 && t < lane); }
        double* sw = reinterpret_cast<double*>(skey);        // (a wave's LDS operations take effect in order)
        if (valid) sw[r] = w;
        const int nvalid = __popcll(__ballot(valid));
        double total = 0.0;
#pragma unroll 8
        for (int t = 0; t < kc; ++t) total = total + sval[t];
        const double target = cfg.top_p * total;
        double cum = 0.0;
        int take = nvalid;
#pragma unroll 8
        for (int t = 0; t < nvalid; ++t) { cum = cum + sw[t]; if (cum >= target) take = min(take, t + 1); }
        if (lane < kc) sflag[lane] = valid && r < take;
      }
    } else {
    // Rank of every valid cluster, stored in place of the flag: sflag = rank+1, 0 = invalid.  The upper halves of the keys
    // decide it but for the clusters that share one: those have the same rank, which two bits a rank show (met once, met
    // again), and only they compare whole keys, and indices.  Weights of zero, many where the scores are far apart, keep one
    // rank for all: they come last and add nothing, so that all are taken or none.  A thread ranks its clusters two at a
    // time, so that a key read serves both.
    // Bound by the pairs: two instructions each, six, four of them on 64 bits, with whole keys throughout; by the two sums
    // below it where the clusters are few.  12 heads x 65 lists of 365 clusters: this kernel 38 -> 30 us; the selection of
    // 30 x 65 lists, 600 clusters 310 -> 182 us, 2 000 clusters 1 546 -> 789, 24 x 65 of 1 171 1 597 -> 726.
    hist[tid] = 0; dup[tid] = 0;                 // 8 192 bits each; the library holds 7 168 clusters
    __syncthreads();
    for (int j = tid; j < kc; j += 512) {
      const int j2 = j + 256;
      const uint32_t k1 = (uint32_t)(skey[j] >> 32);
      int r1 = 0, r2 = 0;
      auto met = [&](int at, int r) __attribute__((always_inline)) {
        if (!sflag[at]) return;
        const int bit = 1 << (r & 31);
        if (sval[at] != 0.0 && (atomicOr(&hist[r >> 5], bit) & bit)) atomicOr(&dup[r >> 5], bit);
        sflag[at] = r + 1;
      };
      if (j2 - lane < kc) {
        const uint32_t k2 = j2 < kc ? (uint32_t)(skey[j2] >> 32) : 0u;
#pragma unroll 8
        for (int t = 0; t < kc; ++t) { const uint32_t kt = (uint32_t)(skey[t] >> 32); r1 += kt > k1; r2 += kt > k2; }
        if (j2 < kc) met(j2, r2);
      } else {
#pragma unroll 8
        for (int t = 0; t < kc; ++t) r1 += (uint32_t)(skey[t] >> 32) > k1;
      }
      met(j, r1);
    }
    __syncthreads();
    for (int j0 = wave * 64; j0 < kc; j0 += 256) {
      const int j = j0 + lane, r = j < kc ? sflag[j] - 1 : -1;
      const bool tie = r >= 0 && sval[j] != 0.0 && ((dup[r >> 5] >> (r & 31)) & 1);
      uint64_t left = __ballot(tie);
      if (__popcll(left) <= 8) {                 // a few: the wave's lanes read the keys for one cluster after the other
        for (; left; left &= left - 1) {
          const int jt = j0 + __builtin_ctzll(left);
          const uint64_t k1 = skey[jt];
          int exact = 0;
          for (int t = lane; t < kc; t += 64) { const uint64_t kt = skey[t]; exact += (kt > k1) || (kt == k1 && t < jt); }
#pragma unroll
          for (int o = 1; o < 64; o <<= 1) exact += __shfl_xor(exact, o);
          if (j == jt) sflag[j] = exact + 1;
        }
      } else if (tie) {
        const uint64_t k1 = skey[j];
        int exact = 0;
#pragma unroll 8
        for (int t = 0; t < kc; ++t) { const uint64_t kt = skey[t]; exact += (kt > k1) || (kt == k1 && t < j); }
        sflag[j] = exact + 1;
      }
    }
    __syncthreads();
    // The weights in rank order go into skey (dead once the ranks are known), then one thread each takes the two sums, chains
    // of rounded adds in a fixed order: the total in ascending index, the running sum in rank order, left in place.  Eight
    // values at a time, the next eight asked for before they are added: only the adds wait for one another.
    double* sw = reinterpret_cast<double*>(skey);
    int nv_local = 0, nz_local = 0;              // clusters, and those with a weight
    for (int j = tid; j < kc; j += 256) { nv_local += sflag[j] != 0; nz_local += sflag[j] != 0 && sval[j] != 0.0; }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) { nv_local += __shfl_xor(nv_local, o); nz_local += __shfl_xor(nz_local, o); }
    if (lane == 0) { wsum[wave] = nv_local; wsum2[wave] = nz_local; }
    __syncthreads();
    const int nvalid = wsum[0] + wsum[1] + wsum[2] + wsum[3], nz = wsum2[0] + wsum2[1] + wsum2[2] + wsum2[3];
    for (int j = tid; j < kc; j += 256) if (sflag[j] && sval[j] != 0.0) sw[sflag[j] - 1] = sval[j];
    __syncthreads();
    auto chain = [&](double* x, int n, auto keep) __attribute__((always_inline)) {
      double sum = 0.0, v[8];
      const int whole = n / 8 * 8;
      if (whole > 0) {
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = x[u];
      }
      for (int j = 0; j < whole; j += 8) {
        double next[8];
        const int ahead = min(j + 8, whole - 8);
#pragma unroll
        for (int u = 0; u < 8; ++u) next[u] = x[ahead + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) { sum = sum + v[u]; if (decltype(keep)::value) x[j + u] = sum; }
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = next[u];
      }
      for (int j = whole; j < n; ++j) { sum = sum + x[j]; if (decltype(keep)::value) x[j] = sum; }
      return sum;
    };
    if (tid == 0) { s_max = cfg.top_p * chain(sval, kc, std::false_type{}); s_take = nvalid; }      // (the maximum has been read)
    if (tid == 64) chain(sw, nz, std::true_type{});
    __syncthreads();
    for (int r0 = wave * 64; r0 < nz; r0 += 256) {
      const uint64_t there = __ballot(r0 + lane < nz && sw[r0 + lane] >= s_max);
      if (there) { if (lane == 0) atomicMin(&s_take, r0 + __builtin_ctzll(there) + 1); break; }
    }
    __syncthreads();
    const int take = s_take;
    for (int j = tid; j < kc; j += 256) sflag[j] = sflag[j] != 0 && sflag[j] <= take;
    }
  }
  __syncthreads();

  // ---- ascending compaction of the selected indices
  int32_t* out = sel_idx + ((size_t)h * cfg.Cq + i) * cfg.cap;
  int run = 0, run_eq = 0, keys = 0;
  const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  for (int j0 = 0; j0 < kc; j0 += 256) {
    const int j = j0 + tid;
    bool f;
    if (use_thr) {
      const bool valid = j < kc && sval[j] > -INFINITY;
      const uint64_t k = j < kc ? skey[j] : 0ull;
      const bool eq = valid && k == thr_key;
      const uint64_t bal_eq = __ballot(eq);
      __syncthreads();
      if (lane == 0) wsum2[wave] = __popcll(bal_eq);
      __syncthreads();
      int eq_before = run_eq + __popcll(bal_eq & lt_mask);
      for (int w = 0; w < wave; ++w) eq_before += wsum2[w];
      run_eq += wsum2[0] + wsum2[1] + wsum2[2] + wsum2[3];
      f = valid && (k > thr_key || (eq && eq_before < thr_rem));
    } else {
      f = j < kc && sflag[j] != 0;
    }
    const uint64_t bal = __ballot(f);
    __syncthreads();
    if (lane == 0) wsum[wave] = __popcll(bal);
    __syncthreads();
    int before = 0;
    for (int w = 0; w < wave; ++w) before += wsum[w];
    if (f) {
      out[run + before + __popcll(bal & lt_mask)] = j;
      if (KEYS) keys += k_sizes[(size_t)h * cfg.cap + j];
    }
    run += wsum[0] + wsum[1] + wsum[2] + wsum[3];
  }
  if (tid == 0) sel_cnt[(size_t)h * cfg.Cq + i] = run;
  if (!KEYS) return;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) keys += __shfl_xor(keys, o);
  __syncthreads();
  if (lane == 0) wsum2[wave] = keys;
  __syncthreads();
  if (tid == 0 && h == 0 && i == 0) sel_keys[(size_t)gridDim.y * cfg.Cq] = 0;
  if (tid == 0) sel_keys[(size_t)h * cfg.Cq + i] = wsum2[0] + wsum2[1] + wsum2[2] + wsum2[3];
}

// Elements of the key tables that the workgroups of select_kernel read in all, up to which they form the scores themselves (one
// key cluster a thread).  A call of 4 x 4 000 tokens, d=128, 65 query clusters, 117 key clusters at most 233 -> 227 us, 16 x 1 800,
// d=64 150 -> 145, 30 x 1 500, d=128 241 -> 236, 1 x 4 096 fp32 206 -> 203; 30 x 4 000, d=64 (15 million) 307 -> 304; past it the
// same time either way (30 x 7 920, 256 clusters, 32 million).
constexpr long long SELECT_SCORES = 16000000;
int launch_select(hipStream_t s, int H, int Cq, int cap, int d, int score_mode, int select_mode, int topk,
                  float top_p, float scale, const float* q_cent, const float* q_mean_norm, const float* k_cent,
                  const float* k_bmin, const float* k_bmax, const int32_t* k_sizes, const int32_t* k_count,
                  const int32_t* full_flag, int32_t* sel_idx, int32_t* sel_cnt, int kc_max, double* scores, int32_t* sel_keys) {
  // kc_max: an upper bound of k_count[h] known to the host; it sizes the LDS arrays (and with
  // them the number of workgroups a CU can hold)
  const int lds_cap = kc_max < cap ? (kc_max + 63) / 64 * 64 : cap;
  SelectCfg c{Cq, cap, d, lds_cap, score_mode, select_mode, topk, (double)top_p, (double)scale};
  const size_t shm = (size_t)lds_cap * 20;
  if (shm > 150 * 1024) return ADACLUSTER_E_BADSHAPE;
  // The kernel's dynamic-LDS limit is raised only when a launch needs more than any launch before it on this
  // device (a call that repeats an earlier shape then consists of launches only, which is what a caller that
  // captures it into a HIP graph needs).
  const int kb = kc_max < cap ? kc_max : cap;
  const bool here = kb <= 256 && (long long)H * Cq * kb * d <= SELECT_SCORES;
  auto launch = [&](auto topp, auto keys, auto dd, auto box) {
    static std::atomic<int> granted[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return ADACLUSTER_E_INTERNAL;
    const auto kernel = select_kernel<decltype(topp)::value, decltype(keys)::value, decltype(dd)::value, decltype(box)::value>;
    if ((int)shm > granted[dev].load()) {
      if (hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm) != hipSuccess)
        return ADACLUSTER_E_INTERNAL;
      granted[dev].store((int)shm);
    }
    kernel<<<dim3(Cq, H), 256, shm, s>>>(c, scores, ScoreTables{q_cent, k_cent, k_bmin, k_bmax}, q_mean_norm, k_sizes, k_count, full_flag, sel_idx, sel_cnt, sel_keys);
    return hipGetLastError() == hipSuccess ? 0 : ADACLUSTER_E_INTERNAL;
  };
  auto select = [&](auto topp, auto keys) {
    using std::integral_constant;
    auto boxes = [&](auto dd) {
      return score_mode == ADACLUSTER_SCORE_BOX ? launch(topp, keys, dd, std::true_type{}) : launch(topp, keys, dd, std::false_type{});
    };
    if (!here) return launch(topp, keys, integral_constant<int, 0>{}, std::false_type{});
    return d == 64 ? boxes(integral_constant<int, 64>{}) : boxes(integral_constant<int, 128>{});
  };
  auto score = [&](auto qg, auto dd, auto box) {
    constexpr int QG = decltype(qg)::value, D = decltype(dd)::value;
    const dim3 g((kb + SCORE_THREADS - 1) / SCORE_THREADS, (Cq + QG - 1) / QG, H);
    score_kernel<QG, D, decltype(box)::value><<<g, SCORE_THREADS, 0, s>>>(c, q_cent, k_cent, k_bmin, k_bmax, k_sizes, k_count, full_flag, scores);
  };
  auto form = [&](auto qg, auto dd) {
    if (score_mode == ADACLUSTER_SCORE_BOX) score(qg, dd, std::true_type{}); else score(qg, dd, std::false_type{});
  };
  auto group = [&](auto qg) {
    if (d == 64) form(qg, std::integral_constant<int, 64>{}); else form(qg, std::integral_constant<int, 128>{});
  };
  // Query clusters a thread: 3 while that leaves every one of the 1024 SIMDs at most a wave (d=128, 5 heads x 110 clusters:
  // 10 us, 5 a thread 13), 13 once it gives every SIMD two, 4 or (boxes, whose rows take twice the registers) 5 in between
  // (12 x 330, d=128: 17 and 20 us, 3 a thread 20 and 25; 30 x 600, d=64: 28 and 31 us, 5 and 4 a thread 34 and 43).
  const long long waves = (long long)((kb + 63) / 64) * H;
  if (here) {}
  else if (waves * ((Cq + 2) / 3) <= 1024) group(std::integral_constant<int, 3>{});
  else if (waves * ((Cq + 12) / 13) >= 2048) group(std::integral_constant<int, 13>{});
  else if (score_mode == ADACLUSTER_SCORE_BOX) group(std::integral_constant<int, 5>{});
  else group(std::integral_constant<int, 4>{});
  auto keys = [&](auto topp) { return sel_keys ? select(topp, std::true_type{}) : select(topp, std::false_type{}); };
  return select_mode == ADACLUSTER_SELECT_TOPP ? keys(std::true_type{}) : keys(std::false_type{});
}

}  // namespace adac
