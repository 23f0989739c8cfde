// Stable label sort (counting sort; one workgroup's LSD radix for short heads) and CSR offsets.
//
// The permutation that groups tokens by cluster label is what makes the centroid
// reduction atomic-free and the K/V gathers cluster-contiguous.  It must be
// deterministic, so ranks inside a segment are taken in item order (wave-wide
// match on the label or digit, never "who won the atomic").
#include "common.h"
#include "launch.h"
#include "small_head.h"
#include <type_traits>

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
// Counting sort of the heads that one workgroup does not hold, two launches or three whatever the number of labels:
//   label_count    one workgroup per segment of CS_ITEMS items: the segment's count of every label;
//   label_columns  exclusive prefix of every label's counts over the segments, and its total (tables of many counts only);
//   label_scatter  a workgroup finds the labels' first positions (every one for itself: from the segments' counts, or m
//                  totals, out of the L2), ranks its items inside the segment and writes them where they belong.  One more
//                  workgroup per head writes what the totals say besides: the CSR offsets and the parts of the centroid
//                  reduction.
// Bound by launch latency and dependent trips to the L2, 4-9 us a launch; items move once.  (Two 7-bit radix passes
// of three launches each, the offsets by binary search in the sorted labels and the parts in a launch of their own were
// eight launches that moved every item and its label twice.  Final key sort of 30 x 75 600 tokens, about 580 labels:
// 69 -> 34 us; 24 x 180 000, about 1 270: 130 -> 53; 12 x 32 760, about 365: 43 -> 20.)
// Eight waves a segment of 2 048, four items a lane, where four waves took eight: most launches here are a workgroup a CU or
// less, and the rank of an item waits for the items before it.  Attention step with one key cluster a list, both of its sorts:
// 30 x 17 550 tokens, 330 labels 98 -> 91 us, 48 x 32 760 222 -> 214, 24 x 180 000 884 -> 869.
// Bins are the labels 0..m-1 and one last bin m for labels outside of that range (a caller's labels of clusters past
// its own count): they stay at the end of the order, where no offset points.  The one-workgroup sort has the same bins.
// ------------------------------------------------------------------------------------------
constexpr int CS_ITEMS = 2048;

__device__ __forceinline__ int label_limit(const int32_t* m_dev, int m_stride, int m_const, int h) {
  return m_dev ? max(0, min(m_dev[(size_t)h * m_stride], m_const)) : m_const;       // (the tables are sized for m_const)
}
template <int WAVES>
__global__ __launch_bounds__(WAVES * 64) void label_count(const int32_t* __restrict__ labels, int N, SortArgs a,
                                                     const int32_t* __restrict__ m_dev, int m_stride, int m_const,
                                                     int nseg, int stride, int32_t* __restrict__ hist) {
  constexpr int CS_NT = WAVES * 64, CS_STEPS = CS_ITEMS / CS_NT;
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
constexpr int CC_WAVES = 4;
__global__ __launch_bounds__(CC_WAVES * 64) void label_columns(SortArgs a, const int32_t* __restrict__ m_dev, int m_stride, int m_const,
                                                       int nseg, int stride, int32_t* __restrict__ hist) {
  const int h = blockIdx.y, lane = threadIdx.x & 63, g = threadIdx.x >> 6, j = blockIdx.x * 64 + lane;
  const int n = head_items(a, h);
  const int m = label_limit(m_dev, m_stride, m_const, h);
  if (n <= 0 || (int)blockIdx.x * 64 > m) return;
  int32_t* hh = hist + (size_t)h * (nseg + 1) * stride + j;
  const int ns = min((n + CS_ITEMS - 1) / CS_ITEMS, nseg), per = (ns + CC_WAVES - 1) / CC_WAVES;
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
  __shared__ int32_t gsum[CC_WAVES][64];
  gsum[g][lane] = run;
  __syncthreads();
  int pos = 0, all = 0;
#pragma unroll
  for (int i = 0; i < CC_WAVES; ++i) { const int v = gsum[i][lane]; if (i < g) pos += v; all += v; }
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

// exclusive prefix of v over the workgroup's threads (w: WAVES integers of LDS, free again after the next barrier)
template <int WAVES>
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
  for (int i = 0; i < WAVES; ++i) { const int u = w[i]; if (i < wave) before += u; total += u; }
  return before + incl - v;
}

template <int WAVES, bool FOLD>
__global__ __launch_bounds__(WAVES * 64) void label_scatter(const int32_t* __restrict__ labels, const int32_t* __restrict__ vals,
                                                       int N, SortArgs a, const int32_t* __restrict__ m_dev, int m_stride,
                                                       int m_const, int nseg, int stride, const int32_t* __restrict__ hist,
                                                       int32_t* __restrict__ perm, int32_t* __restrict__ offs, int offs_stride,
                                                       int32_t* __restrict__ poff, int part_rows, int32_t* __restrict__ pcl,
                                                       int P) {
  constexpr int CS_NT = WAVES * 64, CS_STEPS = CS_ITEMS / CS_NT;
  const int h = blockIdx.y, seg = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (a.active_dev && !a.active_dev[(size_t)h * a.active_stride]) return;
  const int n = head_items(a, h), beg = seg * CS_ITEMS;
  const bool tables = seg == nseg;
  if (!tables && beg >= n) return;
  const int m = label_limit(m_dev, m_stride, m_const, h);
  // LDS, 2 bytes a bin and wave: the first position of every bin (FOLD: and how many items lie in the segments before this
  // one); and then, once every item has taken its own, the waves' counters,
  // two bins a word (items counted, then the next rank inside the segment)
  extern __shared__ int32_t start[];
  const int words = m / 2 + 1;
  uint32_t* const wc = reinterpret_cast<uint32_t*>(start);      // [WAVES][words]
  __shared__ int32_t w0[WAVES], w1[WAVES];
  const int32_t* hh = hist + (size_t)h * (nseg + 1) * stride;
  const int p0 = beg + wave * (CS_ITEMS / WAVES) + lane;
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
  int32_t* const before = start + m + 1;         // FOLD: items of the bin in the segments before this one
  if constexpr (FOLD) {
    const int ns = min((n + CS_ITEMS - 1) / CS_ITEMS, nseg);
    constexpr int BATCH = 12;
    for (int j = tid; j <= m; j += CS_NT) {
      int all = 0, bef = 0;
      for (int sb = 0; sb < ns; sb += BATCH) {
        int c[BATCH];
#pragma unroll
        for (int k = 0; k < BATCH; ++k) c[k] = hh[(size_t)min(sb + k, ns - 1) * stride + j];
#pragma unroll
        for (int k = 0; k < BATCH; ++k) { const int v = sb + k < ns ? c[k] : 0; all += v; if (sb + k < seg) bef += v; }
      }
      start[j] = all; before[j] = bef;
    }
    __syncthreads();
    for (int j = j0; j < j1; ++j) run += start[j];
  } else if (n > 0) {
    for (int j = j0; j < j1; ++j) { const int c = hh[(size_t)nseg * stride + j]; start[j] = c; run += c; }
  }
  int total;
  int base = block_prefix<WAVES>(run, w0, total);
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
    int pb = block_prefix<WAVES>(parts, w1, ptotal);
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
  for (int k = 0; k < CS_STEPS; ++k) first[k] = start[lv[k]] + (FOLD ? before[lv[k]] : hh[(size_t)seg * stride + lv[k]]);
  __syncthreads();
  for (int i = tid; i < WAVES * words; i += CS_NT) wc[i] = 0;
  __syncthreads();
  uint32_t* const mine = wc + wave * words;
#pragma unroll
  for (int k = 0; k < CS_STEPS; ++k) if (p0 + 64 * k < n) atomicAdd(&mine[lv[k] >> 1], 1u << (16 * (lv[k] & 1)));
  __syncthreads();
  for (int i = tid; i < words; i += CS_NT) {
    uint32_t r = 0;                              // (at most CS_ITEMS of a bin: the halves do not meet)
#pragma unroll
    for (int w = 0; w < WAVES; ++w) { const uint32_t c = wc[w * words + i]; wc[w * words + i] = r; r += c; }
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

// LDS of a workgroup of label_scatter (two bytes a bin and wave; the waves' sums of two prefixes), and the most waves whose
// counters stay within the 64 KB that a launch may ask for without further ado.  Bins of one launch: `stride`.
constexpr int MAX_LABELS = 8000;
constexpr int scatter_lds(int waves, int stride) { return 2 * waves * stride + 2 * waves * (int)sizeof(int32_t); }
constexpr int most_waves(int stride) { return scatter_lds(16, stride) <= 65536 ? 16 : scatter_lds(8, stride) <= 65536 ? 8 : 4; }
constexpr int label_bins(int m) { return (m + 1 + 63) / 64 * 64; }
constexpr bool lds_fits() {
  for (int m = 0; m <= MAX_LABELS; ++m)
    if (scatter_lds(most_waves(label_bins(m)), label_bins(m)) > 65536 || 4 * label_bins(m) > 65536) return false;
  return true;
}
static_assert(lds_fits(), "for every number of labels");

int sort_segments(int N) { return (N + CS_ITEMS - 1) / CS_ITEMS; }
size_t sort_table_ints(int N, int m) { return N <= SMALL_ITEMS ? 0 : (size_t)(sort_segments(N) + 1) * label_bins(m); }
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
  const int nseg = sort_segments(n_bound), stride = label_bins(m_bound);
  // dynamic LDS for the bound, so that as many workgroups share a CU as it allows (7 169 bins: 57 KB)
  if (m_bound > MAX_LABELS) return ADACLUSTER_E_INTERNAL;
  auto sort = [&](auto waves, auto fold) {
    constexpr int W = decltype(waves)::value, NT = W * 64;
    constexpr bool FOLD = decltype(fold)::value;
    label_count<W><<<dim3(nseg, H), NT, stride * 4, st>>>(labels, N, a, m_dev, m_stride, m_bound, nseg, stride, sc.hist);
    if (!FOLD) label_columns<<<dim3(stride / 64, H), CC_WAVES * 64, 0, st>>>(a, m_dev, m_stride, m_bound, nseg, stride, sc.hist);
    label_scatter<W, FOLD><<<dim3(nseg + 1, H), NT, 2 * W * stride, st>>>(labels, ulist, N, a, m_dev, m_stride, m_bound, nseg, stride,
                                                                             sc.hist, perm, offs, offs_stride, poff, part_rows, pcl, P);
  };
  // The prefix over the segments inside the scatter, each workgroup for itself, saves a launch (both sorts of the call above:
  // 5 x 9 000 tokens, 64 labels 50 -> 45 us, 12 x 32 760, 1 300 labels 77 -> 76) and reads nseg * stride counts a workgroup: past
  // some 22 000 of them, or 40 segments, the launch is the cheaper one (12 x 32 760, 5 000 labels 88 and 104; 24 x 180 000, 330
  // labels 869 and 884).  Sixteen waves, two items a lane, while that leaves every workgroup a CU to itself: 12 x 32 760, 330
  // labels 75 -> 73, 5 x 9 000 41 -> 40; 48 x 32 760 the other way, 209 and 217.  And no more than have counters in LDS.
  using std::integral_constant;
  const int waves = most_waves(stride);
  if (waves == 4) sort(integral_constant<int, 4>{}, std::false_type{});
  else if (nseg > 40 || nseg * stride > 22000) sort(integral_constant<int, 8>{}, std::false_type{});
  else if (nseg * H > 256 || waves == 8) sort(integral_constant<int, 8>{}, std::true_type{});
  else sort(integral_constant<int, 16>{}, std::true_type{});
  if (poff_done && poff) *poff_done = pcl ? 2 : 1;
  return hipGetLastError() == hipSuccess ? 0 : ADACLUSTER_E_INTERNAL;
}

}  // namespace adac
