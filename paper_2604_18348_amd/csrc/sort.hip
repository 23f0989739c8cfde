// Stable label sort (counting sort; one workgroup's LSD radix for short heads) and CSR offsets.
//
// The permutation that groups tokens by cluster label is what makes the centroid
// reduction atomic-free and the K/V gathers cluster-contiguous.  It must be
// deterministic, so ranks inside a segment are taken in item order (wave-wide
// match on the label or digit, never "who won the atomic").
#include "common.h"
#include "launch.h"
#include "small_head.h"

namespace adac {


struct SortArgs {
  const int32_t* n_dev;  int n_stride;  int n_const;
  const int32_t* active_dev; int active_stride;
};

__device__ __forceinline__ int head_items(const SortArgs& a, int h) {
  if (a.active_dev && !a.active_dev[(size_t)h * a.active_stride]) return 0;   // head not active
  return a.n_dev ? a.n_dev[(size_t)h * a.n_stride] : a.n_const;
}

// ------------------------------------------------------------------------------------------
// Counting sort of the heads that one workgroup does not hold: three launches whatever the number of labels.
//   label_count    one workgroup per segment of CS_ITEMS items: the segment's count of every label;
//   label_columns  exclusive prefix of every label's counts over the segments, and its total;
//   label_scatter  a workgroup turns the totals into the labels' first positions (every one for itself: m integers
//                  out of the L2), ranks its items inside the segment and writes them where they belong.  One more
//                  workgroup per head writes what the totals say besides: the CSR offsets and the parts of the centroid
//                  reduction.
// Bound by launch latency and dependent trips to the L2, 4-7 us a launch; items move once.  (Two 7-bit radix passes
// of three launches each, the offsets by binary search in the sorted labels and the parts in a launch of their own were
// eight launches that moved every item and its label twice.  Final key sort of 30 x 75 600 tokens, about 580 labels:
// 69 -> 34 us; 24 x 180 000, about 1 270: 130 -> 53; 12 x 32 760, about 365: 43 -> 20.)
// Bins are the labels 0..m-1 and one last bin m for labels outside of that range (a caller's labels of clusters past
// its own count): they stay at the end of the order, where no offset points.  The one-workgroup sort has the same bins.
// ------------------------------------------------------------------------------------------
constexpr int CS_ITEMS = 2048, CS_WAVES = 4, CS_NT = CS_WAVES * 64, CS_STEPS = CS_ITEMS / CS_NT;

__device__ __forceinline__ int label_limit(const int32_t* m_dev, int m_stride, int m_const, int h) {
  return m_dev ? max(0, min(m_dev[(size_t)h * m_stride], m_const)) : m_const;       // (the tables are sized for m_const)
}
__global__ __launch_bounds__(CS_NT) void label_count(const int32_t* __restrict__ labels, int N, SortArgs a,
                                                     const int32_t* __restrict__ m_dev, int m_stride, int m_const,
                                                     int nseg, int stride, int32_t* __restrict__ hist) {
  const int h = blockIdx.y, seg = blockIdx.x, tid = threadIdx.x;
  const int n = head_items(a, h), beg = seg * CS_ITEMS;
  if (beg >= n) return;
  const int m = label_limit(m_dev, m_stride, m_const, h);
  extern __shared__ int32_t cnt[];              // m_const + 1
  const int32_t* lab = labels + (size_t)h * N;
  int lv[CS_STEPS];
#pragma unroll
  for (int k = 0; k < CS_STEPS; ++k) { const int p = beg + k * CS_NT + tid; lv[k] = p < n ? lab[p] : 0; }
  for (int j = tid; j <= m; j += CS_NT) cnt[j] = 0;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < CS_STEPS; ++k) if (beg + k * CS_NT + tid < n) atomicAdd(&cnt[label_bin(lv[k], m)], 1);
  __syncthreads();
  int32_t* out = hist + ((size_t)h * (nseg + 1) + seg) * stride;
  for (int j = tid; j <= m; j += CS_NT) out[j] = cnt[j];
}

// 64 labels a workgroup, each wave a quarter of the segments; the counts are read in batches of independent loads,
// first for the wave's total, then again to write the running positions.  Row nseg of the table takes the totals.
__global__ __launch_bounds__(CS_NT) void label_columns(SortArgs a, const int32_t* __restrict__ m_dev, int m_stride, int m_const,
                                                       int nseg, int stride, int32_t* __restrict__ hist) {
  const int h = blockIdx.y, lane = threadIdx.x & 63, g = threadIdx.x >> 6, j = blockIdx.x * 64 + lane;
  const int n = head_items(a, h);
  const int m = label_limit(m_dev, m_stride, m_const, h);
  if (n <= 0 || (int)blockIdx.x * 64 > m) return;
  int32_t* hh = hist + (size_t)h * (nseg + 1) * stride + j;
  const int ns = min((n + CS_ITEMS - 1) / CS_ITEMS, nseg), per = (ns + CS_WAVES - 1) / CS_WAVES;
  const int s0 = min(ns, g * per), s1 = min(ns, s0 + per);
  const bool mine = j <= m;
  constexpr int BATCH = 12;
  int run = 0;
  for (int sb = s0; sb < s1; sb += BATCH) {
    int c[BATCH];
#pragma unroll
    for (int k = 0; k < BATCH; ++k) c[k] = mine && sb + k < s1 ? hh[(size_t)(sb + k) * stride] : 0;
#pragma unroll
    for (int k = 0; k < BATCH; ++k) run += c[k];
  }
  __shared__ int32_t gsum[CS_WAVES][64];
  gsum[g][lane] = run;
  __syncthreads();
  int pos = 0, all = 0;
#pragma unroll
  for (int i = 0; i < CS_WAVES; ++i) { const int v = gsum[i][lane]; if (i < g) pos += v; all += v; }
  if (g == 0 && mine) hh[(size_t)nseg * stride] = all;
  for (int sb = s0; sb < s1; sb += BATCH) {
    int c[BATCH];
#pragma unroll
    for (int k = 0; k < BATCH; ++k) c[k] = mine && sb + k < s1 ? hh[(size_t)(sb + k) * stride] : 0;
#pragma unroll
    for (int k = 0; k < BATCH; ++k) {
      if (mine && sb + k < s1) hh[(size_t)(sb + k) * stride] = pos;
      pos += c[k];
    }
  }
}

// exclusive prefix of v over the workgroup's threads (w: CS_WAVES integers of LDS, free again after the next barrier)
__device__ __forceinline__ int block_prefix(int v, int32_t* w, int& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) { const int u = __shfl_up(incl, o); if (lane >= o) incl += u; }
  if (lane == 63) w[wave] = incl;
  __syncthreads();
  int before = 0;
  total = 0;
#pragma unroll
  for (int i = 0; i < CS_WAVES; ++i) { const int u = w[i]; if (i < wave) before += u; total += u; }
  return before + incl - v;
}

__global__ __launch_bounds__(CS_NT) void label_scatter(const int32_t* __restrict__ labels, const int32_t* __restrict__ vals,
                                                       int N, SortArgs a, const int32_t* __restrict__ m_dev, int m_stride,
                                                       int m_const, int nseg, int stride, const int32_t* __restrict__ hist,
                                                       int32_t* __restrict__ perm, int32_t* __restrict__ offs, int offs_stride,
                                                       int32_t* __restrict__ poff, int part_rows, int32_t* __restrict__ pcl,
                                                       int P) {
  const int h = blockIdx.y, seg = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (a.active_dev && !a.active_dev[(size_t)h * a.active_stride]) return;
  const int n = head_items(a, h), beg = seg * CS_ITEMS;
  const bool tables = seg == nseg;
  if (!tables && beg >= n) return;
  const int m = label_limit(m_dev, m_stride, m_const, h);
  // LDS, 8 bytes a bin: the first position of every bin; and then, once every item has taken its own, the waves' counters,
  // two bins a word (items counted, then the next rank inside the segment)
  extern __shared__ int32_t start[];
  const int words = m / 2 + 1;
  uint32_t* const wc = reinterpret_cast<uint32_t*>(start);      // [CS_WAVES][words]
  __shared__ int32_t w0[CS_WAVES], w1[CS_WAVES];
  const int32_t* hh = hist + (size_t)h * (nseg + 1) * stride;
  const int p0 = beg + wave * (CS_ITEMS / CS_WAVES) + lane;
  int lv[CS_STEPS], vv[CS_STEPS];
  if (!tables) {
#pragma unroll
    for (int k = 0; k < CS_STEPS; ++k) {
      const int p = p0 + 64 * k;
      lv[k] = p < n ? label_bin(labels[(size_t)h * N + p], m) : m;
      vv[k] = p < n ? (vals ? vals[(size_t)h * N + p] : p) : 0;
    }
  }
  // bins tid * per .. of this thread (no items: every bin is empty, the table holds nothing)
  const int per = (m + 1 + CS_NT - 1) / CS_NT, j0 = min(m + 1, tid * per), j1 = min(m + 1, j0 + per);
  int run = 0;
  if (n > 0) for (int j = j0; j < j1; ++j) { const int c = hh[(size_t)nseg * stride + j]; start[j] = c; run += c; }
  int total;
  int base = block_prefix(run, w0, total);
  for (int j = j0; j < j1; ++j) { const int c = n > 0 ? start[j] : 0; start[j] = base; base += c; }
  __syncthreads();
  if (tables) {
    int32_t* of = offs + (size_t)h * offs_stride;
    for (int j = tid; j <= m; j += CS_NT) of[j] = start[j];
    if (!poff) return;
    // poff[j]: parts of the clusters before j (a cluster of c rows has ceil(c / part_rows)); pcl[b]: cluster of part b,
    // written when there are more than 128 clusters (with fewer, the reduction finds its cluster by a vote)
    int32_t* po = poff + (size_t)h * offs_stride;
    int32_t* pc = pcl && m > 128 ? pcl + (size_t)h * P : nullptr;
    const int q1 = min(m, j1);
    int parts = 0;
    for (int j = j0; j < q1; ++j) parts += (start[j + 1] - start[j] + part_rows - 1) / part_rows;
    int ptotal;
    int pb = block_prefix(parts, w1, ptotal);
    for (int j = j0; j < q1; ++j) {
      po[j] = pb;
      const int np = (start[j + 1] - start[j] + part_rows - 1) / part_rows;
      if (pc) for (int q = 0; q < np && pb + q < P; ++q) pc[pb + q] = j;
      pb += np;
    }
    if (tid == 0) po[m] = ptotal;
    return;
  }
  // where the segment's first item of this item's bin goes
  int first[CS_STEPS];
#pragma unroll
  for (int k = 0; k < CS_STEPS; ++k) first[k] = start[lv[k]] + hh[(size_t)seg * stride + lv[k]];
  __syncthreads();
  for (int i = tid; i < CS_WAVES * words; i += CS_NT) wc[i] = 0;
  __syncthreads();
  uint32_t* const mine = wc + wave * words;
#pragma unroll
  for (int k = 0; k < CS_STEPS; ++k) if (p0 + 64 * k < n) atomicAdd(&mine[lv[k] >> 1], 1u << (16 * (lv[k] & 1)));
  __syncthreads();
  for (int i = tid; i < words; i += CS_NT) {
    uint32_t r = 0;                              // (at most CS_ITEMS of a bin: the halves do not meet)
#pragma unroll
    for (int w = 0; w < CS_WAVES; ++w) { const uint32_t c = wc[w * words + i]; wc[w * words + i] = r; r += c; }
  }
  __syncthreads();
  const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  const int bits = 32 - __clz(m | 1);
  volatile uint32_t* next = mine;                // touched by this wave only from here on, in program order
  int32_t* ph = perm + (size_t)h * N;
#pragma unroll
  for (int k = 0; k < CS_STEPS; ++k) {
    const bool valid = p0 + 64 * k < n;
    const int b = lv[k], sh = 16 * (b & 1);
    // lanes holding my bin: intersect, bit by bit, the ballots of lanes that agree with me
    uint64_t same = __ballot(valid);
    for (int i = 0; i < bits; ++i) {
      const bool bit = (b >> i) & 1;
      const uint64_t bal = __ballot(bit);
      same &= bit ? bal : ~bal;
    }
    const int rank = __popcll(same & lt_mask);
    const int pos = first[k] + (int)((next[b >> 1] >> sh) & 0xFFFFu) + rank;
    __builtin_amdgcn_wave_barrier();
    if (valid && rank == 0) atomicAdd(&mine[b >> 1], (uint32_t)__popcll(same) << sh);
    __builtin_amdgcn_wave_barrier();
    if (valid) ph[pos] = vv[k];
  }
}

// One workgroup per head: see sort_one_head.
__global__ __launch_bounds__(1024) void sort_small(const int32_t* __restrict__ labels, const int32_t* __restrict__ vals_in,
                                                   int N, int scratch, int passes, SortArgs a, const int32_t* __restrict__ m_dev,
                                                   int m_stride, int m_const, int32_t* __restrict__ lab_a,
                                                   int32_t* __restrict__ val_a, int32_t* __restrict__ lab_b,
                                                   int32_t* __restrict__ perm, int32_t* __restrict__ offs,
                                                   int offs_stride, int32_t* __restrict__ poff, int part_rows) {
  const int h = blockIdx.x;
  if (a.active_dev && !a.active_dev[(size_t)h * a.active_stride]) return;
  const int n = head_items(a, h);
  const int m = label_limit(m_dev, m_stride, m_const, h);
  const size_t o = (size_t)h * N, so = (size_t)h * scratch;
  sort_one_head(labels + o, vals_in ? vals_in + o : nullptr, n, passes, m, lab_a + so, val_a + so, lab_b + so, perm + o,
                offs + (size_t)h * offs_stride, poff ? poff + (size_t)h * offs_stride : nullptr, part_rows);
}

int sort_segments(int N) { return (N + CS_ITEMS - 1) / CS_ITEMS; }
size_t sort_table_ints(int N, int m) { return N <= SMALL_ITEMS ? 0 : (size_t)(sort_segments(N) + 1) * ((m + 1 + 63) / 64 * 64); }
int sort_scratch_ints(int N) { return min(N, SMALL_ITEMS); }

int launch_sort(hipStream_t st, int H, int N, int n_bound, int m_bound,
                const int32_t* labels, const int32_t* ulist,
                const int32_t* n_dev, int n_stride, const int32_t* m_dev, int m_stride,
                const int32_t* active_dev, int active_stride,
                int32_t* perm, int32_t* offs, int offs_stride, const SortScratch& sc, int32_t* poff,
                int part_rows, int32_t* pcl, int P, int* poff_done, int foreign) {
  SortArgs a{n_dev, n_stride, n_bound, active_dev, active_stride};
  if (poff_done) *poff_done = 0;
  if (n_bound <= SMALL_ITEMS) {
    int bits = 1;
    while ((1 << bits) < m_bound + (foreign ? 1 : 0)) ++bits;       // (the digits of the last bin too)
    const int passes = (bits + RBITS - 1) / RBITS;
    sort_small<<<H, 1024, 0, st>>>(labels, ulist, N, sort_scratch_ints(N), passes, a, m_dev, m_stride, m_bound, sc.lab_a, sc.val_a, sc.lab_b,
                                   perm, offs, offs_stride, poff, part_rows);
    if (poff_done && poff) *poff_done = 1;
    return hipGetLastError() == hipSuccess ? 0 : ADACLUSTER_E_INTERNAL;
  }
  const int nseg = sort_segments(n_bound), stride = (m_bound + 1 + 63) / 64 * 64;
  // dynamic LDS for the bound, so that as many workgroups share a CU as it allows (7 169 bins: 57 KB)
  if (m_bound > 8000) return ADACLUSTER_E_INTERNAL;
  label_count<<<dim3(nseg, H), CS_NT, stride * 4, st>>>(labels, N, a, m_dev, m_stride, m_bound, nseg, stride, sc.hist);
  label_columns<<<dim3(stride / 64, H), CS_NT, 0, st>>>(a, m_dev, m_stride, m_bound, nseg, stride, sc.hist);
  label_scatter<<<dim3(nseg + 1, H), CS_NT, stride * 8 + 64, st>>>(labels, ulist, N, a, m_dev, m_stride, m_bound, nseg, stride,
                                                                   sc.hist, perm, offs, offs_stride, poff, part_rows, pcl, P);
  if (poff_done && poff) *poff_done = pcl ? 2 : 1;
  return hipGetLastError() == hipSuccess ? 0 : ADACLUSTER_E_INTERNAL;
}

}  // namespace adac
