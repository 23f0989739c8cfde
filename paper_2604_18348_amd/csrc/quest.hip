// Quest scores between query rows and key pages (Sec. 3.2.3): the upper bound of Eq. 1 evaluated
// with plain vector arithmetic, and its reformulation as two matrix products (Eq. 2, Algorithm 2)
// on the matrix cores.  Both take the per-dimension maxima R+ and minima R- of every page (for a
// single vector per page, e.g. a cluster centroid, Algorithm 2 uses R+ = max(k, 0), R- = min(k, 0):
// `clamp` does that on the fly from one tensor).
//   S[h, i, j] = sum_d max(q_d R+_jd, q_d R-_jd)                       (Eq. 1)
//              = sum_d max(q_d, 0) R+_jd + sum_d min(q_d, 0) R-_jd     (Eq. 2)
#include "common.h"
#include "launch.h"

#include <type_traits>

namespace adac {

// ---- Eq. 1 with vector arithmetic: 16 TI x 64 outputs per workgroup, TI x 4 per thread, operands staged through
// LDS 32 dimensions at a time, a dimension's values of all rows side by side, so that a thread reads four at once.
// Bound by vector issue: max(q p, q n) is q times the larger of p and n where q >= 0, and times the smaller where q < 0 (rounding is
// monotonic), so a term is a select and a multiply-add behind one comparison of q for four pages, not two products, a maximum and an
// add: 2.25 instructions of 4.  That holds while no product overflows, which values below 2^63 rule out (a multiply-add does not round its product
// to infinity); from the first 32 dimensions with any other on, a workgroup forms its terms as Eq. 1 writes them.  18 heads x 12 039 rows x 865 pages, d=128, bf16 1 949 -> 1 181 us, 6 x 81 444 x 416, d=128, fp32 2 344 -> 1 451, 8 x 75 861 x
// 387, d=64 1 375 -> 917, 10 x 168 x 105 17.6 -> 9.8 (56 % of the vector rate; 4 x 4 outputs a thread, scalar LDS reads: 57 % for 4 a term).
template <typename T, int TI>
__global__ __launch_bounds__(256) void quest_alu(int Lq, int Lk, int d, int clamp, int aligned, int whole, const T* __restrict__ Q,
                                                 const T* __restrict__ Rp, const T* __restrict__ Rn,
                                                 float* __restrict__ S) {
  constexpr int TD = 32, QR = 16 * TI, E = 16 / sizeof(T), PIECES = TD / E;      // E: values of a 16-byte piece
  __shared__ __attribute__((aligned(16))) float qs[TD][QR + 4], his[TD][68], los[TD][68];
  __shared__ int odd;
  constexpr float PLAIN = 0x1p63f;
  const int h = blockIdx.z, q0 = blockIdx.x * QR, k0 = blockIdx.y * 64, tid = threadIdx.x;
  const int tq = (tid >> 4) * TI, tk = (tid & 15) * 4;
  const T* Qh = Q + (size_t)h * Lq * d;
  const T* Ph = Rp + (size_t)h * Lk * d;
  const T* Nh = Rn + (size_t)h * Lk * d;
  float acc[TI][4];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;
  auto piece = [&](const T* p, float (&x)[E]) __attribute__((always_inline)) {
    T raw[E];
    if (whole) *reinterpret_cast<uint4*>(raw) = *reinterpret_cast<const uint4*>(p);
    else {                                         // (a caller's tensors may start anywhere)
#pragma unroll
      for (int e = 0; e < E; ++e) raw[e] = p[e];
    }
#pragma unroll
    for (int e = 0; e < E; ++e) x[e] = Elem<T>::load(&raw[e]);
  };
  if (tid == 0) odd = 0;
  for (int d0 = 0; d0 < d; d0 += TD) {
    __syncthreads();                               // the values of the step before have been read
    bool small = true;
    for (int e = tid; e < QR * PIECES; e += 256) {
      const int r = e % QR, g = e / QR;
      float x[E] = {};
      if (q0 + r < Lq) piece(Qh + (size_t)(q0 + r) * d + d0 + g * E, x);
#pragma unroll
      for (int i = 0; i < E; ++i) { qs[g * E + i][r] = x[i]; small = small && fabsf(x[i]) < PLAIN; }
    }
    for (int e = tid; e < 64 * PIECES; e += 256) {
      const int r = e % 64, g = e / 64;
      float p[E] = {}, n[E] = {};
      if (k0 + r < Lk) {
        piece(Ph + (size_t)(k0 + r) * d + d0 + g * E, p);
        piece(Nh + (size_t)(k0 + r) * d + d0 + g * E, n);
      }
#pragma unroll
      for (int i = 0; i < E; ++i) {
        if (clamp) { p[i] = fmaxf(p[i], 0.f); n[i] = fminf(n[i], 0.f); }
        const float hi = fmaxf(p[i], n[i]), lo = fminf(p[i], n[i]);
        his[g * E + i][r] = hi; los[g * E + i][r] = lo;
        small = small && fabsf(hi) < PLAIN && fabsf(lo) < PLAIN;
      }
    }
    if (!small) odd = 1;                           // (stays: the steps that follow are formed term by term as well)
    __syncthreads();
    auto terms = [&](auto plain) __attribute__((always_inline)) {
#pragma unroll 4
      for (int cc = 0; cc < TD; ++cc) {
        float q[TI];
        if constexpr (TI == 2) *reinterpret_cast<float2*>(q) = *reinterpret_cast<const float2*>(&qs[cc][tq]);
        else {
#pragma unroll
          for (int i = 0; i < TI; i += 4) *reinterpret_cast<float4*>(q + i) = *reinterpret_cast<const float4*>(&qs[cc][tq + i]);
        }
        float hi[4], lo[4];
        *reinterpret_cast<float4*>(hi) = *reinterpret_cast<const float4*>(&his[cc][tk]);
        *reinterpret_cast<float4*>(lo) = *reinterpret_cast<const float4*>(&los[cc][tk]);
#pragma unroll
        for (int i = 0; i < TI; ++i) {
          const bool neg = q[i] < 0.f;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            if constexpr (decltype(plain)::value) acc[i][j] = fmaf(q[i], neg ? lo[j] : hi[j], acc[i][j]);
            else acc[i][j] += fmaxf(q[i] * hi[j], q[i] * lo[j]);
          }
        }
      }
    };
    if (__builtin_amdgcn_readfirstlane(odd)) terms(std::false_type{}); else terms(std::true_type{});
  }
  float* Sh = S + (size_t)h * Lq * Lk;
#pragma unroll
  for (int i = 0; i < TI; ++i) {
    if (q0 + tq + i >= Lq) break;
    float* row = Sh + (size_t)(q0 + tq + i) * Lk + k0 + tk;
    if (aligned) {                                 // pages in fours, rows that start at 16 bytes
      if (k0 + tk < Lk) *reinterpret_cast<float4*>(row) = float4{acc[i][0], acc[i][1], acc[i][2], acc[i][3]};
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) if (k0 + tk + j < Lk) row[j] = acc[i][j];
    }
  }
}

// A bf16 value is negative where it is negative as a 16-bit integer: two packed integer operations per pair.
typedef short s16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void split_signs(uint4& pos, uint4& neg) {
  uint32_t* a = reinterpret_cast<uint32_t*>(&pos);
  uint32_t* b = reinterpret_cast<uint32_t*>(&neg);
  const s16x2_t zero = {0, 0};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    a[i] = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2_t, a[i]), zero));
    b[i] = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(s16x2_t, b[i]), zero));
  }
}

template <int D, int NW>
__global__ __launch_bounds__(NW * 64) void quest_mfma(int Lq, int Lk, int clamp, const bf16raw* __restrict__ Q,
                                                      const bf16raw* __restrict__ Rp, const bf16raw* __restrict__ Rn,
                                                      float* __restrict__ S) {
  constexpr int KS = D / 16, CH = D / 8, NT = NW * 64, ROWB = D * 2, QB = 32 * ROWB;
  constexpr int LOADS = KS > NW ? KS / NW : 1;            // direct-to-LDS loads a loading wave issues per query block
  // rows of span + 8 floats: a store of the accumulator layout touches two rows 4 apart, and 4 rows are 32 banks away
  constexpr int SPAN = NW * 32, STRIDE = SPAN + 8;
  __shared__ __attribute__((aligned(16))) char qs[3 * QB];
  __shared__ __attribute__((aligned(16))) float ts[32 * STRIDE];
  const int h = blockIdx.z, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 31, hb = lane >> 5;
  // More pages than the span: a workgroup row of the grid computes `SPAN` pages, of which a score row writes those of
  // the lines that start inside all but the last 32; the next one starts there.
  const int k0 = blockIdx.y * (SPAN - 32);
  const bool single = Lk <= SPAN, last = k0 + SPAN >= Lk;
  const int nblocks = (Lq + 31) / 32;
  const int b0 = (int)((long long)nblocks * blockIdx.x / gridDim.x), b1 = (int)((long long)nblocks * (blockIdx.x + 1) / gridDim.x);
  if (b0 >= b1) return;

  // chunk q of row r sits in slot q ^ swz(r) of its LDS row: operand reads free of bank conflicts
  auto swz = [](int r) __attribute__((always_inline)) { return D == 128 ? (r & 15) : ((r >> 1) & 7); };
  const char* Qh = (const char*)(Q + (size_t)h * Lq * D);
  const uint32_t qs0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)qs;
  const bool loads = wave < KS;                           // (KS kilobytes a block, one per load)
  auto issue = [&](int slot, int b) __attribute__((always_inline)) {     // rows past the end repeat the last one
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int item = (wave * LOADS + i) * 64 + lane, r = item / CH;
      dma_b128(qs0 + slot * QB + (wave * LOADS + i) * 1024,
               Qh + (size_t)min(b * 32 + r, Lq - 1) * ROWB + (((item % CH) ^ swz(r)) * 16));
    }
  };
  if (loads) { issue(0, b0); issue(1, b0 + 1); }
  bf16x8_t P[KS], N[KS];
  {
    const size_t r = ((size_t)h * Lk + min(k0 + wave * 32 + c, Lk - 1)) * D + hb * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      uint4 up = *reinterpret_cast<const uint4*>(Rp + r + ks * 16), un = *reinterpret_cast<const uint4*>(Rn + r + ks * 16);
      if (clamp) split_signs(up, un);
      P[ks] = *reinterpret_cast<const bf16x8_t*>(&up);
      N[ks] = *reinterpret_cast<const bf16x8_t*>(&un);
    }
  }
  int qaddr[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) qaddr[ks] = c * ROWB + (((ks * 2 + hb) ^ swz(c)) * 16);
  wait_vmcnt<0>();
  lds_barrier();
  // Scores wait in LDS so that a 16-byte piece of LDS is an aligned one of S.  One span: the rows follow one another as they
  // do in S, `mis` floats behind the start (a block is a multiple of 128 bytes: the same for every block of a head).  More:
  // row r is moved by (mis + r * Lk) % 4 floats.  A float a lane was four
  // times the store instructions and a walk over rows and pages: 2 x 75 600 rows, 450 pages, d=64 58 -> 53 us (5.1 TB/s),
  // 3 x 50 001 x 333 48 -> 39, 4 x 17 776 x 200, d=128 23.5 -> 21.0, 1 x 180 000 x 60 16.6 -> 14.6; more spans: 24 x 9 000 x
  // 700, d=128 187 -> 171, 2 x 75 600 x 993 180 -> 169, 1 x 100 000 x 513, its second span one page, 62.4 -> 63.2.
  // (Whole lines as streaming stores: the call alone 0.92 of its time over 16 shapes on three buffers in turn, 2 x 75 600 x 450 62 -> 58 us,
  // but what reads the scores next reads them from memory: call and a reader of all scores 1.09, 2 x 75 600 x 450 143 -> 151, 4 x 76 823 x
  // 352, d=128 224 -> 254, on one buffer 1.06; and 4 x 32 760 x 300, d=64 on one buffer, without a reader, 31 -> 40.)
  const int mis = (int)((uintptr_t)(S + (size_t)h * Lq * Lk) >> 2) & 3;
  const int stores = single ? 8 * Lk / NT : 0;            // store instructions a wave issues per whole block, at least
  int slot = 0;
  for (int b = b0; b < b1; ++b) {
    if (loads) issue(slot >= 1 ? slot - 1 : 2, b + 2);    // the slot of block b - 1, which every wave has read
    const char* q = qs + slot * QB;
    f32x16_t acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      uint4 pos = *reinterpret_cast<const uint4*>(q + qaddr[ks]), neg = pos;
      split_signs(pos, neg);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8_t*>(&pos), P[ks], acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8_t*>(&neg), N[ks], acc, 0, 0, 0);
    }
    lds_barrier();                                        // the scores of block b - 1 have left LDS
    // value v of the tile is query 8*(v/4) + 4*hb + v%4 of the block, page slot wave*32 + c
    if (!single) {
      float* tw = ts + 4 * hb * STRIDE + wave * 32 + c;
#pragma unroll
      for (int v = 0; v < 16; ++v) tw[(8 * (v >> 2) + (v & 3)) * STRIDE + ((mis + (v & 3) * Lk) & 3)] = acc[v];
    } else if (wave * 32 + c < Lk) {
      float* tw = ts + mis + 4 * hb * Lk + wave * 32 + c;
#pragma unroll
      for (int v = 0; v < 16; ++v) tw[(8 * (v >> 2) + (v & 3)) * Lk] = acc[v];
    }
    // the rows of block b + 1 have landed: younger than their request are the stores of block b - 1 and the request above
    if (loads) { if (stores >= 3) wait_vmcnt<3 + LOADS>(); else if (stores == 2) wait_vmcnt<2 + LOADS>(); else wait_vmcnt<LOADS>(); }
    lds_barrier();
    float* Sb = S + ((size_t)h * Lq + (size_t)b * 32) * Lk;
    const int nrows = min(32, Lq - b * 32);
    // floats [from, to) of a run that starts at `at` in LDS and in S, first .. first + 3 this lane's of the first step
    auto leave = [&](const float* at, float* out, int from, int to, int first, int step) __attribute__((always_inline)) {
      for (int e = first; e < to; e += step) {
        const float4 v = *reinterpret_cast<const float4*>(at + e);
        if (e >= from && e + 4 <= to) {
          *reinterpret_cast<float4*>(out + e) = v;
        } else {
          const float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int i = 0; i < 4; ++i) if (e + i >= from && e + i < to) out[e + i] = x[i];
        }
      }
    };
    if (single) {                 // whole rows: one run over all of them
      leave(ts, Sb - mis, mis, mis + nrows * Lk, 4 * tid, 4 * NT);
    } else {
      for (int r = wave; r < nrows; r += NW) {
        float* row = Sb + (size_t)r * Lk;
        // first page at or after p that starts a line of S
        auto line = [&](int p) __attribute__((always_inline)) { return p + (int)((0u - (uint32_t)((uintptr_t)(row + p) >> 2)) & 31u); };
        const int from = k0 == 0 ? 0 : line(k0), to = last ? Lk : line(k0 + SPAN - 32), mr = (mis + r * Lk) & 3;
        leave(ts + r * STRIDE, row + k0 - mr, from - k0 + mr, to - k0 + mr, ((from - k0 + mr) & ~3) + 4 * lane, 256);
      }
    }
    slot = slot == 2 ? 0 : slot + 1;
  }
  wait_vmcnt<0>();       // nothing of this wave is still on its way to LDS when it ends
}

int launch_quest_scores(hipStream_t s, int dtype, int form, int clamp, int H, int Lq, int Lk, int d, const void* Q,
                        const void* Rp, const void* Rn, float* S) {
  if (form == 0) {
    const int aligned = Lk % 4 == 0 && ((uintptr_t)S & 15) == 0, whole = (((uintptr_t)Q | (uintptr_t)Rp | (uintptr_t)Rn) & 15) == 0;
    auto go = [&](auto ti, auto type) {
      constexpr int TI = decltype(ti)::value;
      using T = decltype(type);
      quest_alu<T, TI><<<dim3((Lq + 16 * TI - 1) / (16 * TI), (Lk + 63) / 64, H), 256, 0, s>>>(Lq, Lk, d, clamp, aligned, whole, (const T*)Q, (const T*)Rp, (const T*)Rn, S);
    };
    auto rows = [&](auto type) {
      const long long tiles = (long long)((Lk + 63) / 64) * H;
      // Eight rows a thread while that leaves eight workgroups a CU (6 x 25 053 x 177, d=128 224 us, four 235; 13 x 8 192 x 111, d=64,
      // 1 664 workgroups, 65.6 and 62.7), two where four leave less than two a CU: a workgroup's own chain is the launch then (1 x 4 213 x
      // 207, d=128 21.1 us, four 31.1, eight 42.7).
      if (tiles * ((Lq + 127) / 128) >= 2048) go(std::integral_constant<int, 8>{}, type);
      else if (tiles * ((Lq + 63) / 64) >= 512) go(std::integral_constant<int, 4>{}, type);
      else go(std::integral_constant<int, 2>{}, type);
    };
    if (dtype == ADACLUSTER_BF16) rows(bf16raw{}); else rows(float{});
  } else {
    if (dtype != ADACLUSTER_BF16) return ADACLUSTER_E_UNSUPPORTED;
    // One page tile a wave and no more waves than the pages fill, up to 16: with four waves for 60 pages 1 x 180 000 rows
    // took 24 us, with two 17.  The grid is what the chip holds at once (bounded by LDS and registers), every workgroup
    // with an equal run of query blocks, because a workgroup loads its pages once.
    const int nw = Lk <= 64 ? 2 : Lk <= 128 ? 4 : Lk <= 256 ? 8 : 16, span = nw * 32;
    const int resident = 256 * (nw >= 8 ? 16 / nw : nw == 4 ? 3 : d == 64 ? 6 : 4);
    const int spans = Lk <= span ? 1 : 1 + (Lk - span + span - 33) / (span - 32);
    const int nblocks = (Lq + 31) / 32;
    const long long per = resident / ((long long)H * spans);
    const dim3 g((unsigned)(per < 1 ? 1 : per > nblocks ? nblocks : per), spans, H);
    auto go = [&](auto kernel) {
      kernel<<<g, nw * 64, 0, s>>>(Lq, Lk, clamp, (const bf16raw*)Q, (const bf16raw*)Rp, (const bf16raw*)Rn, S);
    };
    if (d == 64) { if (nw == 2) go(quest_mfma<64, 2>); else if (nw == 4) go(quest_mfma<64, 4>); else if (nw == 8) go(quest_mfma<64, 8>); else go(quest_mfma<64, 16>); }
    else { if (nw == 2) go(quest_mfma<128, 2>); else if (nw == 4) go(quest_mfma<128, 4>); else if (nw == 8) go(quest_mfma<128, 8>); else go(quest_mfma<128, 16>); }
  }
  return hipGetLastError() == hipSuccess ? 0 : ADACLUSTER_E_INTERNAL;
}

// ------------------------------------------------------------------------------------------
// Matrix-core probe: every wave runs four independent chains of v_mfma_f32_32x32x16_bf16 on operands that
// never leave its registers.  It moves no data, so the rate it reaches is the bf16 MFMA throughput the chip
// sustains at the clock it holds under that load: the yardstick quoted beside the published peak.
// ------------------------------------------------------------------------------------------
static constexpr int PROBE_BLOCKS = 2048, PROBE_THREADS = 256, PROBE_CHAINS = 4;
__global__ __launch_bounds__(PROBE_THREADS) void mfma_probe(int iters, float* __restrict__ sink) {
  const int tid = threadIdx.x;
  bf16x8_t a, b;
#pragma unroll
  for (int i = 0; i < 8; ++i) { a[i] = (__bf16)(float)((tid + i) & 3); b[i] = (__bf16)(float)((tid >> 2) & 1); }
  f32x16_t c[PROBE_CHAINS];
#pragma unroll
  for (int j = 0; j < PROBE_CHAINS; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) c[j][v] = 0.f;
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int j = 0; j < PROBE_CHAINS; ++j) c[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c[j], 0, 0, 0);
  }
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < PROBE_CHAINS; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) s += c[j][v];
  if (blockIdx.x == 0) sink[tid] = s;
}

int launch_mfma_probe(hipStream_t s, int iters, float* sink, size_t sink_floats, double* flops) {
  if (sink_floats < (size_t)PROBE_THREADS) return ADACLUSTER_E_BADARG;
  mfma_probe<<<PROBE_BLOCKS, PROBE_THREADS, 0, s>>>(iters, sink);
  *flops = (double)PROBE_BLOCKS * (PROBE_THREADS / 64) * (double)iters * PROBE_CHAINS * (2.0 * 32 * 32 * 16);
  return hipGetLastError() == hipSuccess ? 0 : ADACLUSTER_E_INTERNAL;
}

}  // namespace adac
