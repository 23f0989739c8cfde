// k-means building blocks for the query clustering (Sec. 3.1, Alg. 3 line 1) and the
// multi-stage key clustering (Algorithm 1):
//   * point-to-centre assignment as an MFMA GEMM  C . X^T  with an in-lane running arg-max
//     (bf16 I/O) or a plain fp32 kernel (fp32 I/O);
//   * atomic-free centroid update: segmented sums over the label-sorted token order;
//   * the stage bookkeeping of Algorithm 1 (centre count rule, threshold filter, compaction
//     of the unassigned set U), kept on the device.
#include "common.h"
#include "launch.h"

#include <type_traits>

namespace adac {

// ------------------------------------------------------------------------------------------
// assignment
// ------------------------------------------------------------------------------------------
// modes: 0 = fixed (row_off 0, m = m_const, n = N, every head)
//        1 = stage (row_off = ccount, m = m_t, n = ucount, only active heads)
//        2 = final (row_off 0, m = ccount, n = N, every head)
//        3 = final, seeded (bf16): only the centres of the stages after the first are visited (row_off =
//            stage_offs[1], m = ccount - row_off); every point starts from its best first-stage centre, whose
//            label and score the last pass of stage 0 left in seed_lab / seed_score (that pass ran over all
//            points against exactly those centres).  Labels are indices into all centres, as in mode 2.
// keep_lab / keep_score (stage 0, last pass): a second copy of the labels and the best score, for mode 3.
struct AssignCfg {
  int mode; int m_const; int N; int cap;
  const KState* st; const int32_t* ulist;
  int32_t* keep_lab; float* keep_score;
  const int32_t* seed_lab; const float* seed_score;
  const float* tau; int32_t* keep_cnt; int keep_stride;   // points of this workgroup that the threshold leaves in U (a late
                                                          // stage's last pass): keep_cnt[h * keep_stride + workgroup]
  double* dist_sum;                                       // sum of the distances of this workgroup's points (the first stage's last
                                                          // pass, for tau): dist_sum[h * gridDim.x + workgroup]
                                                          // (assign_rows: of this wave's points, for both)
  int32_t* surv; int32_t* stage_of; int stage;            // stage_pass, with keep_cnt (or NULL): the survivors themselves, from where the
                                                          // workgroup's points start, and the stage of the points that leave U
};
constexpr int PASS_POINTS = 256;        // points of a workgroup of stage_pass (twice that where it combines)
constexpr int ASSIGN_POINTS_LP = 256, ASSIGN_POINTS_F32 = 64;     // points of an assignment workgroup

__device__ __forceinline__ bool assign_setup(const AssignCfg& c, int h, int& n, int& m, int& row_off) {
  if (c.mode == 0) { n = c.N; m = c.m_const; row_off = 0; return true; }
  const KState& s = c.st[h];
  if (c.mode == 1) { n = s.ucount; m = s.m_t; row_off = s.ccount; return s.active != 0; }
  if (c.mode == 3) { n = c.N; row_off = s.stage_offs[1]; m = s.ccount - row_off; return true; }
  n = c.N; m = s.ccount; row_off = 0; return true;
}

// score(x, c) = x.c + bias(c), bias = -||c||^2/2 (Euclidean arg-min) or 0 (cosine arg-max);
// label = arg-max, ties to the lowest index;  dist2 = ||x||^2 - 2 score.
//
// MFMA formulation: D[32 centres x 32 points] += A[32 x 16] B[16 x 32] with A = centre rows from
// LDS and B = point rows held in registers for the whole kernel.  In the 32x32 accumulator a lane
// owns ONE point (column lane%32) and 16 centres, so the arg-max over centres runs in-lane; the
// two half-waves are merged once at the end.  Two workgroups per CU in the launch bounds keep the
// register budget at 256, so the accumulators are ordinary VGPRs that the arg-max reads directly (with
// 512 the compiler parks them in AGPRs and copies every value out first).
constexpr int ACC_MAXM = 128;          // most centres that member sums on the matrix cores are kept for (qpass_mfma, stage_pass)

typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4_t;
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;
typedef __attribute__((address_space(3))) void lds_void_t;

template <int D>
__global__ __launch_bounds__(256, 2) void assign_mfma(const bf16raw* __restrict__ X, AssignCfg cfg,
                                                                const bf16raw* __restrict__ cent,
                                                                const float* __restrict__ bias,
                                                                int32_t* __restrict__ labels, float* __restrict__ dist2) {
  constexpr int CB = D == 128 ? 64 : 128;   // centres per LDS chunk (16 KB either way; larger chunks measured slower)
  constexpr int KS = D / 16;
  constexpr int PB = 2;                 // 32-point blocks per wave
  constexpr int CROWB = D * 2, CH = D / 8;  // bytes and 16-byte pieces of a centre row
  const int h = blockIdx.y;
  int n, m, row_off;
  if (!assign_setup(cfg, h, n, m, row_off)) return;
  const int base = blockIdx.x * (4 * PB * 32);
  if (base >= n) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 31, hb = lane >> 5;

  // Centre chunks go global -> LDS directly (no registers), one chunk ahead, in two buffers that are LDS
  // objects of their own (the compiler orders an LDS read behind an outstanding direct load only when
  // both may touch the same object, so the load of chunk i+1 runs under the arithmetic of chunk i).
  // Rows are unpadded; piece g of row r sits in slot g ^ swz(r), which keeps the 16-byte operand
  // reads of 16 consecutive rows in 16 different bank groups.
  __shared__ __attribute__((aligned(16))) char cs0[CB * CROWB];
  __shared__ __attribute__((aligned(16))) char cs1[CB * CROWB];
  __shared__ __attribute__((aligned(16))) float bs0[CB];
  __shared__ __attribute__((aligned(16))) float bs1[CB];
  auto swz = [](int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); };

  // B operand: this lane's point rows
  bf16x8_t xf[PB][KS];
  float xn2[PB];
  int pos[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
    pos[pb] = base + wave * (PB * 32) + pb * 32 + c;
    float ss = 0.f;
    if (pos[pb] < n) {
      const int tok = cfg.ulist ? cfg.ulist[(size_t)h * cfg.N + pos[pb]] : pos[pb];
      const bf16raw* row = X + ((size_t)h * cfg.N + tok) * D + hb * 8;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const uint4 raw = *reinterpret_cast<const uint4*>(row + ks * 16);
        xf[pb][ks] = *reinterpret_cast<const bf16x8_t*>(&raw);
      }
      if (dist2) {                       // ||x||^2 is only needed for the distances
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const uint4 raw = *reinterpret_cast<const uint4*>(&xf[pb][ks]);
          const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float a = __uint_as_float(w[q] << 16), b = __uint_as_float(w[q] & 0xFFFF0000u);
            ss = fmaf(a, a, ss); ss = fmaf(b, b, ss);
          }
        }
      }
    } else {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) { const uint4 z = {0, 0, 0, 0}; xf[pb][ks] = *reinterpret_cast<const bf16x8_t*>(&z); }
    }
    xn2[pb] = ss + __shfl_xor(ss, 32);
  }

  // Running arg-max with the position inside a 32x32 accumulator tile carried in the low 4
  // mantissa bits of the score (a 2^-19 relative perturbation, far below the near-tie margin):
  // one and-or per value, then a max3 tree, then one compare per tile.
  float best[PB]; int btile[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) { best[pb] = -INFINITY; btile[pb] = 0; }
  // Seeded final pass: the half-wave that owns the seed centre's accumulator position starts from the seed,
  // in the packed form a visit of that centre would have left (score with the position code in the low bits);
  // a negative tile marks "still the seed".
  int slab[PB];
  const int label_base = cfg.mode == 3 ? row_off : 0;
  if (cfg.seed_lab) {
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
      slab[pb] = 0;
      if (pos[pb] < n) {
        const int j0 = cfg.seed_lab[(size_t)h * cfg.N + pos[pb]];
        const float s0 = cfg.seed_score[(size_t)h * cfg.N + pos[pb]];
        const int r = j0 & 31, v0 = ((r >> 3) << 2) | (r & 3);
        slab[pb] = j0;
        if (hb == ((r >> 2) & 1)) {
          best[pb] = __uint_as_float((__float_as_uint(s0) & 0xFFFFFFF0u) | (uint32_t)(15 - v0));
          btile[pb] = -1;
        }
      }
    }
    if (m <= 0) {                      // no later stage: the first-stage labels are final
#pragma unroll
      for (int pb = 0; pb < PB; ++pb)
        if (hb == 0 && pos[pb] < n) labels[(size_t)h * cfg.N + pos[pb]] = slab[pb];
      return;
    }
  }

  const bf16raw* ch = cent + ((size_t)h * cfg.cap + row_off) * D;
  const float* bh = bias + (size_t)h * cfg.cap + row_off;

  // operand addresses inside a chunk (bytes), fixed for the whole kernel
  int kaddr[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) kaddr[ks] = c * CROWB + (((ks * 2 + hb) ^ swz(c)) * 16);
  // thread -> (row, slot) of its pieces of a chunk; rows past m repeat the last centre (their bias never wins)
  constexpr int PT = CB * CH / 256;
  auto issue_chunk = [&](int c0, char* dst_base) {
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const int item = tid + i * 256;
      const int r = item / CH, sl = item % CH;
      const int row = min(c0 + r, m - 1);
      const char* src = reinterpret_cast<const char*>(ch) + (size_t)row * CROWB + ((sl ^ swz(r)) * 16);
      const int dst = (wave * 64 + i * 256) * 16;     // wave-uniform; the lane offset is implicit
      __builtin_amdgcn_global_load_lds(src, (lds_void_t*)(dst_base + dst), 16, 0, 0);
    }
  };
  auto load_bias = [&](int c0) { return (tid < CB && c0 + tid < m) ? bh[c0 + tid] : -3.0e38f; };   // finite: survives the bit packing
  auto compute_chunk = [&](int c0, const char* cs, const float* bs) {
    const int rbmax = min(CB / 32, (m - c0 + 31) / 32);
    for (int rb = 0; rb < rbmax; ++rb) {
      f32x16_t acc[PB];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float4 b4 = *reinterpret_cast<const float4*>(&bs[rb * 32 + 8 * i + 4 * hb]);
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
          acc[pb][4 * i + 0] = b4.x; acc[pb][4 * i + 1] = b4.y;
          acc[pb][4 * i + 2] = b4.z; acc[pb][4 * i + 3] = b4.w;
        }
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(cs + rb * 32 * CROWB + kaddr[ks]);
#pragma unroll
        for (int pb = 0; pb < PB; ++pb)
          acc[pb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, xf[pb][ks], acc[pb], 0, 0, 0);
      }
      const int tile_id = (c0 >> 5) + rb;
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) {
        float pk[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) pk[v] = __uint_as_float((__float_as_uint(acc[pb][v]) & 0xFFFFFFF0u) | (uint32_t)(15 - v));
        float tm = fmaxf(fmaxf(pk[0], pk[1]), pk[2]);
#pragma unroll
        for (int v = 3; v < 15; v += 2) tm = fmaxf(fmaxf(tm, pk[v]), pk[v + 1]);
        tm = fmaxf(tm, pk[15]);
        if (tm > best[pb]) { best[pb] = tm; btile[pb] = tile_id; }
      }
    }
  };
  // one step: request the next chunk, work on this one, then let the request land
  auto step = [&](int c0, const char* cs, const float* bs, char* csn, float* bsn) {
    const bool more = c0 + CB < m;
    float bnext = 0.f;
    if (more) { bnext = load_bias(c0 + CB); issue_chunk(c0 + CB, csn); }
    compute_chunk(c0, cs, bs);
    if (more && tid < CB) bsn[tid] = bnext;
    __builtin_amdgcn_s_waitcnt(0x0F70);     // vmcnt(0): this wave's pieces of the next chunk are in LDS
    __syncthreads();
  };
  {
    const float b0 = load_bias(0);
    issue_chunk(0, cs0);
    if (tid < CB) bs0[tid] = b0;
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
  }
  for (int c0 = 0; c0 < m; c0 += 2 * CB) {
    step(c0, cs0, bs0, cs1, bs1);
    if (c0 + CB < m) step(c0 + CB, cs1, bs1, cs0, bs0);
  }
  int kept = 0;
  double dsum = 0.0;
  const bool counts = cfg.keep_cnt && dist2;
  const float t2 = counts ? cfg.tau[1] : 0.f;
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
    // accumulator value v of a tile is centre  32*tile + 8*(v/4) + 4*hb + v%4
    const int v = 15 - (int)(__float_as_uint(best[pb]) & 15u);   // 15-v was packed: equal scores >= 0 go to the lowest centre
    int bidx = label_base + btile[pb] * 32 + 8 * (v >> 2) + 4 * hb + (v & 3);
    if (cfg.seed_lab && btile[pb] < 0) bidx = slab[pb];
    float bv = __uint_as_float(__float_as_uint(best[pb]) & 0xFFFFFFF0u);
    const float ob = __shfl_xor(bv, 32);
    const int oi = __shfl_xor(bidx, 32);
    if (ob > bv || (ob == bv && oi < bidx)) { bv = ob; bidx = oi; }
    const float d2 = fmaxf(xn2[pb] - 2.f * bv, 0.f);
    if (counts) kept += __popcll(__ballot(hb == 0 && pos[pb] < n && !(d2 < t2)));
    if (hb == 0 && pos[pb] < n) {
      if (cfg.dist_sum) dsum += (double)sqrtf(d2);
      labels[(size_t)h * cfg.N + pos[pb]] = bidx;
      if (dist2) dist2[(size_t)h * cfg.N + pos[pb]] = d2;
      if (cfg.keep_lab) { cfg.keep_lab[(size_t)h * cfg.N + pos[pb]] = bidx; cfg.keep_score[(size_t)h * cfg.N + pos[pb]] = bv; }
    }
  }
  if (counts) {
    __shared__ int32_t wkept[4];
    if (lane == 0) wkept[wave] = kept;
    __syncthreads();
    if (tid == 0) cfg.keep_cnt[(size_t)h * cfg.keep_stride + blockIdx.x] = wkept[0] + wkept[1] + wkept[2] + wkept[3];
  }
  if (cfg.dist_sum) {
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) dsum += __shfl_xor(dsum, o);      // (the upper half-wave holds zeros)
    __shared__ double wsum[4];
    if (lane == 0) wsum[wave] = dsum;
    __syncthreads();
    if (tid == 0) cfg.dist_sum[(size_t)h * gridDim.x + blockIdx.x] = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
  }
}

// ------------------------------------------------------------------------------------------
// Opening a stage of Algorithm 1: what stage_open, the opening form of stage_pass and kstages_small share
// ------------------------------------------------------------------------------------------
struct OpenCfg {
  int N, cap, n_max, m0, m_min, max_stages, u_min;
  int first;                       // the first stage opens: no filter, U is every token (`in` is not read)
  int items, nblk, cnt_stride;     // points per count; workgroups that move survivors
  const KState* in; KState* out;
  const float* dist2; const float* tau; const int32_t* cnt;
  const int32_t* uin; int32_t* uout; const int32_t* surv; int32_t* stage_of; int stage;      // `stage`: the one that ends
  int32_t* sums; int32_t* report; int epoch;   // [4] device counters, zero between launches (`first` clears them); host slot
  void* lp; float* f32; float* bias;
};

struct NewState { int ucount, ccount, m_t, stage, done, full, active; };      // a state without its tables

// Where in a list of n points initial centre j of m is: floor((2j+1) n / 2m).
__device__ __forceinline__ int sample_at(int j, int n, int m) {
  const uint64_t p = (2ull * j + 1) * (uint32_t)n;
  return (2ull * m * (uint32_t)n) >> 32 ? (int)(p / (2u * m)) : (int)((uint32_t)p / (2u * m));
}

// Head of the while-loop: done?  flag F?  else the number of centres.
__device__ __forceinline__ void loop_head(NewState& s, int N, int n_max, int m0, int m_min, int max_stages, int u_min) {
  if (s.ucount == 0) s.done = 1;
  else if (s.ccount >= n_max) { s.full = 1; s.done = 1; }
  else if (s.stage >= max_stages || s.ucount <= u_min) s.done = 1;
  s.active = !s.done;
  if (s.active) {
    const uint64_t p = (uint64_t)m0 * (uint32_t)s.ucount + (uint32_t)(N - 1);
    const int m = p >> 32 ? (int)(p / (uint32_t)N) : (int)((uint32_t)p / (uint32_t)N);      // (a division of 64 bits is a microsecond)
    s.m_t = min(max(m_min, min(m0, m)), s.ucount);
  } else s.m_t = 0;
}

// By one thread of a head: the last head to report writes {active heads, max |U|, max m_t, epoch} to the host's slot.
__device__ __forceinline__ void report_stage(const OpenCfg& c, const NewState& s, bool act) {
  if (!c.report) return;
  // Atomics alone, each waited for where the next may not overtake it: a fence instead writes back and drops what the launch has in the L2.
  const auto done = [] { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
  if (act) { atomicAdd(&c.sums[0], 1); atomicMax(&c.sums[1], s.ucount); atomicMax(&c.sums[2], s.m_t); }
  done();
  if (atomicAdd(&c.sums[3], 1) == (int)gridDim.y - 1) {
    int v[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) v[i] = atomicExch(&c.sums[i], 0);
    atomicExch(&c.sums[3], 0);
#pragma unroll
    for (int i = 0; i < 3; ++i) __hip_atomic_store(&c.report[i], v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    done();
    __hip_atomic_store(&c.report[3], c.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);     // (the host polls this word)
  }
}

// By one workgroup of a head, which has no points (the report waits for memory several times): the state of a head that was closed before goes on as it is ...
__device__ __forceinline__ void carry_state(const OpenCfg& c, int h, int tid) {
  if (tid < (int)(sizeof(KState) / 4)) reinterpret_cast<int32_t*>(&c.out[h])[tid] = reinterpret_cast<const int32_t*>(&c.in[h])[tid];
  if (tid == 0) report_stage(c, NewState{}, false);
}
// ... and the new state of one that was not is written and reported.
__device__ __forceinline__ void write_state(const OpenCfg& c, int h, int tid, const NewState& s) {
  if (tid == 0) {
    KState& o = c.out[h];
    o.ucount = s.ucount; o.ccount = s.ccount; o.m_t = s.m_t; o.stage = s.stage; o.done = s.done; o.full = s.full;
    o.active = s.active; o.pad = 0;
    report_stage(c, s, s.active);
  }
  if (tid <= ADACLUSTER_MAX_STAGES) {
    const int i = tid;
    c.out[h].stage_offs[i] = c.first ? 0 : i == s.stage ? s.ccount : c.in[h].stage_offs[i];
    c.out[h].u_hist[i] = c.first ? (i == 0 ? c.N : 0) : i == s.stage ? s.ucount : c.in[h].u_hist[i];
  }
}

// Survivors by position: the last pass of a stage left them, in order, from the start of every `items` points on, and their
// counts.  OPEN_COUNTS counts at most.  Every wave forms the prefix for itself, of counts `lane` and 64 + `lane`, and all write the same:
// no barrier.  Returns the number of survivors; pre[k] of the counts behind nb is that number.
constexpr int OPEN_COUNTS = STAGE_SUM_BLOCKS;
__device__ __forceinline__ int survivor_prefix(int nb, int c0, int c1, int32_t* pre /* LDS, [OPEN_COUNTS + 1] */) {
  const int lane = threadIdx.x & 63;
  static_assert(OPEN_COUNTS == 128, "two counts a lane");
  int a = lane < nb ? c0 : 0, b = lane + 64 < nb ? c1 : 0;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(a, o), v = __shfl_up(b, o);
    if (lane >= o) { a += u; b += v; }
  }
  const int first = __builtin_amdgcn_readlane(a, 63);
  if (lane == 0) pre[0] = 0;
  pre[lane + 1] = a;
  pre[lane + 65] = first + b;
  __builtin_amdgcn_wave_barrier();
  return first + __builtin_amdgcn_readlane(b, 63);
}
// Where in the list of a head survivors p[0 .. K-1] are: the searches side by side, their reads of a step together.
template <int K>
__device__ __forceinline__ void survivors_at(const int32_t* pre, int items, int (&p)[K]) {
  int lo[K];
#pragma unroll
  for (int k = 0; k < K; ++k) lo[k] = 0;
#pragma unroll
  for (int o = OPEN_COUNTS / 2; o >= 1; o >>= 1) {
    int v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = pre[lo[k] + o];
#pragma unroll
    for (int k = 0; k < K; ++k) lo[k] += v[k] <= p[k] ? o : 0;
  }
#pragma unroll
  for (int k = 0; k < K; ++k) p[k] += lo[k] * items - pre[lo[k]];
}

// A value that is the same in every lane, for the compiler too.  What is read from LDS counts as different from lane to lane, and a
// branch or loop on it around a barrier as one that lanes may take apart.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// The opening of a stage by every workgroup (x) of a head (y) for itself: its points, centres and where those go, and the survivors'
// prefix.  False: the head is done.  The last workgroup, behind those that may have points, writes and reports the state: the first
// one's points waited for that, 2-4 us.
__device__ __forceinline__ bool open_stage(const OpenCfg& oc, int h, int32_t* pre, int& n, int& m, int& row_off) {
  const int tid = threadIdx.x, lane = tid & 63;
  const bool writes = blockIdx.x == gridDim.x - 1;
  NewState s{oc.N, 0, 0, 0, 0, 0, 0};
  if (oc.first) {
    if (oc.sums && h == 0 && blockIdx.x == 0 && tid < 4) oc.sums[tid] = 0;
  } else {
    const KState& o = oc.in[h];
    const int32_t* cnt = oc.cnt + (size_t)h * oc.cnt_stride;          // (ahead of the state: one trip for both)
    const int c0 = cnt[min(lane, oc.cnt_stride - 1)], c1 = cnt[min(lane + 64, oc.cnt_stride - 1)];
    if (!o.active) {
      if (writes) carry_state(oc, h, tid);
      return false;
    }
    const int nb = min((int)((uint32_t)(min(o.ucount, oc.N) + oc.items - 1) / (uint32_t)oc.items), OPEN_COUNTS);
    s.ccount = o.ccount + o.m_t; s.stage = o.stage + 1; s.full = o.full;
    s.ucount = survivor_prefix(nb, c0, c1, pre);
  }
  loop_head(s, oc.N, oc.n_max, oc.m0, oc.m_min, oc.max_stages, oc.u_min);
  if (writes) { write_state(oc, h, tid, s); return false; }
  if (!s.active) return false;
  n = s.ucount; m = s.m_t; row_off = s.ccount;
  return true;
}

struct PassSums { float* psum; int32_t* bcnt; int P; int nb_stride; };
constexpr int STAGE_COUNTS = 128;      // counts of a block in PassSums::bcnt
// Sum of columns 4 cl .. 4 cl + 3 over the members of centre j, from the blocks in their order, and the number of members.  By
// the D / 4 lanes of a centre together.
template <int D>
__device__ __forceinline__ float4 block_sum(const PassSums& prev, int h, int j, int nb, int cl, int& nj) {
  constexpr int LPC = D / 4, BATCH = 8;
  nj = 0;
  for (int b = cl; b < nb; b += LPC) nj += prev.bcnt[((size_t)h * prev.nb_stride + b) * STAGE_COUNTS + j];
  const float* ps = prev.psum + ((size_t)h * prev.P + (size_t)j * prev.nb_stride) * D + cl * 4;
  float4 s = {0.f, 0.f, 0.f, 0.f};
  for (int b0 = 0; b0 < nb; b0 += BATCH) {
    float4 t[BATCH];
#pragma unroll
    for (int u = 0; u < BATCH; ++u) t[u] = *reinterpret_cast<const float4*>(ps + (size_t)min(b0 + u, nb - 1) * D);
#pragma unroll
    for (int u = 0; u < BATCH; ++u) if (b0 + u < nb) { s.x += t[u].x; s.y += t[u].y; s.z += t[u].z; s.w += t[u].w; }
  }
#pragma unroll
  for (int o = 1; o < LPC; o <<= 1) nj += __shfl_xor(nj, o);
  return s;
}
// The sums of the R waves that share a tile of 32 centres, waves ct * R .. ct * R + R - 1, to the rows of block b of centres below m.  All
// waves hand theirs over at once and every thread adds pieces of the result, ((0+4)+(2+6))+((1+5)+(3+7)) of eight waves: two barriers
// (half of the waves to the other half, until one holds all, six: 1.3 and, d=128, 2.4 us, now 0.7 and 1.3).
// `ps`: LDS that is free behind a barrier, [NW][32][D] floats: piece q (16 bytes) of row r sits in slot q ^ (r & 7).
template <int D, int NW>
__device__ __forceinline__ void store_sums(const f32x16_t (&sacc)[D / 32], float* ps, const PassSums& out, int h, int b, int m, int R, int wave, int c, int hb) {
  constexpr int DT = D / 32, PPR = D / 4;
  __syncthreads();                       // the points have been read
#pragma unroll
  for (int db = 0; db < DT; ++db)
#pragma unroll
    for (int i = 0; i < 4; ++i)          // value v of a tile is dim db*32 + 8*(v/4) + 4*hb + v%4 of its centre c
      *reinterpret_cast<float4*>(ps + (size_t)(wave * 32 + c) * D + ((db * 8 + 2 * i + hb) ^ (c & 7)) * 4) =
          float4{sacc[db][4 * i], sacc[db][4 * i + 1], sacc[db][4 * i + 2], sacc[db][4 * i + 3]};
  __syncthreads();
  for (int item = threadIdx.x; item < m * PPR; item += NW * 64) {
    const int j = item / PPR, q = item % PPR, r = j & 31;
    const float* at = ps + (size_t)((j >> 5) * R * 32 + r) * D + (q ^ (r & 7)) * 4;
    const auto part = [&](int k) __attribute__((always_inline)) { return *reinterpret_cast<const float4*>(at + (size_t)k * 32 * D); };
    const auto add = [](float4 a, float4 b) __attribute__((always_inline)) { return float4{a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w}; };
    float4 v;
    if (R == 8) v = add(add(add(part(0), part(4)), add(part(2), part(6))), add(add(part(1), part(5)), add(part(3), part(7))));
    else if (R == 4) v = add(add(part(0), part(2)), add(part(1), part(3)));
    else if (R == 2) v = add(part(0), part(1));
    else v = part(0);
    *reinterpret_cast<float4*>(out.psum + ((size_t)h * out.P + (size_t)j * out.nb_stride + b) * D + q * 4) = v;
  }
}

// ------------------------------------------------------------------------------------------
// A pass of a stage of Algorithm 1 with at most ACC_MAXM centres (bf16): assignment and member sums together.
// ------------------------------------------------------------------------------------------
// A workgroup is NW waves of 64 points.  The scores and their in-lane arg-max are those of assign_mfma, the centres all in
// LDS.  An update pass (`out`) then leaves, per centre, the sum and the count of the workgroup's points that chose it, so
// that the update needs neither a label sort nor a segmented reduction: a second product, S^T[32 dims x 32 centres] +=
// X^T[32 dims x 16 points] . E[16 points x 32 centres] with E the one-hot label matrix: exact products, fp32 accumulation
// in a fixed order.  Block b of head h writes row j * nb_stride + b of the head's part-sum table for centre j, and
// bcnt[(h * nb_stride + b) * ACC_MAXM + j].  The last pass leaves squared distances, and what the filter wants to know.
// COMBINE: the centres are not read but formed here, from what the update pass before left (`prev`), by every workgroup for
// itself; the head's first one writes them out.  That takes the place of a launch of finalize_centroids, 5-6 us of latency
// each, where a head's sums are small enough to be read by all of its workgroups (combine_fits): of a stage of 12 x 4 000
// points, d=128, two passes and two launches between them, 9.5 + 6 us each, are two of 12 and 14, and the last pass with its
// launch, 6 + 5.5, one of 10; a call of 12 x 32 760 tokens 880 -> 863 us, of 5 x 9 247 tokens 572 -> 561.  (With the sums and
// the list of points asked for ahead of the state the same; sixteen sums in flight at d=64 spill: 13 -> 25 us.)
// OPEN: the first pass of a stage does what stage_open does, in its place.  The last pass of the stage before (keep_count behind
// the first stage) has left its survivors as a list, from the start of every `items` points on, with their counts: every
// workgroup sums the counts, knows |U|, the loop's decision and m_t, and finds its points and the centres by position.  Latency
// bound: two trips to the L2 more than a pass whose list and centres lie ready, where the launch had five (30 x 5 000 points,
// d=64: 8 + 8.5 -> 12 us; key clusterings of 30 x 7 920 tokens 170 -> 153 us, 12 x 25 500 208 -> 198, 30 x 17 776 570 -> 550).
enum PassCentres { PASS_READ, PASS_COMBINE, PASS_OPEN };
template <int D, int NW, int FORM>
__global__ __launch_bounds__(NW * 64, D == 64 ? 4 : 2) void stage_pass(const bf16raw* __restrict__ X, AssignCfg cfg, bf16raw* __restrict__ cent,
                                                      float* __restrict__ cent_f32, float* __restrict__ bias,
                                                      float* __restrict__ dist2, PassSums prev, PassSums out, OpenCfg oc) {
  constexpr int KS = D / 16, PB = 2, CROWB = D * 2, CH = D / 8, DT = D / 32, NT = NW * 64;
  const int h = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 31, hb = lane >> 5, base = blockIdx.x * NT;
  int n, m, row_off;
  __shared__ int32_t pre[FORM == PASS_OPEN ? OPEN_COUNTS + 1 : 1];
  int pos[PB], tok[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) pos[pb] = base + wave * (PB * 32) + pb * 32 + c;
  if constexpr (FORM == PASS_OPEN) {
    if (!open_stage(oc, h, pre, n, m, row_off)) return;
  } else {
    // (the points are asked for with the state, and those past the last one, whatever stands there, forgotten: one trip for both)
    if (cfg.ulist) {
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) tok[pb] = cfg.ulist[(size_t)h * cfg.N + min(pos[pb], cfg.N - 1)];
    }
    if (!assign_setup(cfg, h, n, m, row_off)) return;
  }
  if (base >= n) return;
  m = min(m, ACC_MAXM);
  const int CT = (m + 31) >> 5;
  // The centres, then the points, then the partial sums of the waves.  Piece g (16 bytes) of centre row r sits in slot g ^
  // swz(r), of point row r in slot g ^ xswz(r) (see qpass_mfma).
  __shared__ __attribute__((aligned(16))) char pool[NT * CROWB];
  __shared__ __attribute__((aligned(16))) float bs[ACC_MAXM];
  __shared__ __attribute__((aligned(16))) int32_t lab_s[NT];
  __shared__ int32_t cnt_s[ACC_MAXM];
  static_assert(NT >= ACC_MAXM, "the centres fit the buffer of the points");
  auto swz = [](int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); };
  auto xswz = [](int r) { return D == 128 ? (((r & 3) << 2) | ((r >> 2) & 3)) : ((((r >> 1) & 1) << 2) | (((r >> 1) & 7) >> 1)); };

  // B operand: this lane's point rows (one of any for points past the last one)
  bf16x8_t xf[PB][KS];
  // (opening: centre j is survivor floor((2j+1) n / 2m); looked up with the points, so that all rows are then asked for together)
  __shared__ int32_t ctok[FORM == PASS_OPEN ? ACC_MAXM : 1];
  if constexpr (FORM == PASS_OPEN) {
    static_assert(PB == 2, "two points and a centre a thread");
    const int q = sample_at(min(tid, m - 1), n, m);
    int at[3] = {min(pos[0], n - 1), min(pos[1], n - 1), q};
    if (!oc.first) {
      survivors_at(pre, oc.items, at);
#pragma unroll
      for (int k = 0; k < 3; ++k) at[k] = oc.surv[(size_t)h * cfg.N + at[k]];
    }
    tok[0] = at[0]; tok[1] = at[1];
    if (tid < m) ctok[tid] = at[2];
    __syncthreads();
  } else {
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) tok[pb] = pos[pb] >= n ? 0 : cfg.ulist ? tok[pb] : pos[pb];
  }
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
    const bf16raw* row = X + ((size_t)h * cfg.N + tok[pb]) * D + hb * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uint4 raw = *reinterpret_cast<const uint4*>(row + ks * 16);
      xf[pb][ks] = *reinterpret_cast<const bf16x8_t*>(&raw);
    }
  }
  const size_t crow = (size_t)h * cfg.cap + row_off;
  if constexpr (FORM == PASS_OPEN) {
    // CH lanes a centre, a piece of its row each.  The head's first workgroup writes the centres out, and each its part of U, for
    // the passes behind
    if (!oc.first && hb == 0) {
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) if (pos[pb] < n) oc.uout[(size_t)h * cfg.N + pos[pb]] = tok[pb];
    }
    const int sl = tid % CH;
#pragma unroll 4
    for (int j = tid / CH; j < CT * 32; j += NT / CH) {
      uint4 r = {0u, 0u, 0u, 0u};
      if (j < m) r = *reinterpret_cast<const uint4*>(X + ((size_t)h * cfg.N + ctok[j]) * D + sl * 8);
      const uint32_t w[4] = {r.x, r.y, r.z, r.w};
      float img[8], ss = 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        img[2 * q] = __uint_as_float(w[q] << 16); img[2 * q + 1] = __uint_as_float(w[q] & 0xFFFF0000u);
        ss = fmaf(img[2 * q], img[2 * q], ss); ss = fmaf(img[2 * q + 1], img[2 * q + 1], ss);
      }
#pragma unroll
      for (int o = 1; o < CH; o <<= 1) ss += __shfl_xor(ss, o);
      *reinterpret_cast<uint4*>(pool + j * CROWB + ((sl ^ swz(j)) * 16)) = r;
      if (sl == 0) bs[j] = j < m ? -0.5f * ss : -3.0e38f;      // (rows past the last centre: zeros under a bias that never wins)
      if (blockIdx.x == 0 && j < m) {
        const size_t at = (crow + j) * D + sl * 8;
        *reinterpret_cast<uint4*>(cent + at) = r;
        *reinterpret_cast<float4*>(cent_f32 + at) = float4{img[0], img[1], img[2], img[3]};
        *reinterpret_cast<float4*>(cent_f32 + at + 4) = float4{img[4], img[5], img[6], img[7]};
        if (sl == 0) bias[crow + j] = -0.5f * ss;
      }
    }
  } else if constexpr (FORM == PASS_COMBINE) {
    // LPC lanes a centre, four columns each; the blocks' sums in block order
    constexpr int LPC = D / 4;
    const int cl = tid % LPC, nb = (n + NT - 1) / NT;
    for (int j = tid / LPC; j < CT * 32; j += NT / LPC) {
      uint2 r = {0u, 0u};
      float bj = -3.0e38f;                               // (rows past the last centre: zeros under a bias that never wins)
      if (j < m) {
        int nj;
        const float4 s = block_sum<D>(prev, h, j, nb, cl, nj);
        const size_t at = (crow + j) * D + cl * 4;
        if (nj > 0) {
          const float cnt = (float)nj;
          const bf16raw v0 = f32_to_bf16(s.x / cnt), v1 = f32_to_bf16(s.y / cnt), v2 = f32_to_bf16(s.z / cnt), v3 = f32_to_bf16(s.w / cnt);
          const float4 img = {bf16_to_f32(v0), bf16_to_f32(v1), bf16_to_f32(v2), bf16_to_f32(v3)};
          r = uint2{(uint32_t)v0 | ((uint32_t)v1 << 16), (uint32_t)v2 | ((uint32_t)v3 << 16)};
          float ss = fmaf(img.x, img.x, 0.f);
          ss = fmaf(img.y, img.y, ss); ss = fmaf(img.z, img.z, ss); ss = fmaf(img.w, img.w, ss);
#pragma unroll
          for (int o = 1; o < LPC; o <<= 1) ss += __shfl_xor(ss, o);
          bj = -0.5f * ss;
          if (blockIdx.x == 0) {
            *reinterpret_cast<uint2*>(cent + at) = r;
            *reinterpret_cast<float4*>(cent_f32 + at) = img;
            if (cl == 0) bias[crow + j] = bj;
          }
        } else {                                         // an empty cluster keeps its centre
          r = *reinterpret_cast<const uint2*>(cent + at);
          bj = bias[crow + j];
        }
      }
      *reinterpret_cast<uint2*>(pool + j * CROWB + (((cl >> 1) ^ swz(j)) * 16) + (cl & 1) * 8) = r;
      if (cl == 0) bs[j] = bj;
    }
  } else {
#pragma unroll
    for (int i = 0; i < ACC_MAXM * CH / NT; ++i) {         // whole tiles, all in flight; rows past m repeat the last centre
      const int item = tid + i * NT, r = item / CH, sl = item % CH;
      if (r < CT * 32)
        dma_b128((uint32_t)(uintptr_t)(lds_void_t*)pool + (wave * 64 + i * NT) * 16,
                 reinterpret_cast<const char*>(cent + (crow + min(r, m - 1)) * D) + ((sl ^ swz(r)) * 16));
    }
    if (tid < CT * 32) bs[tid] = tid < m ? bias[crow + tid] : -3.0e38f;      // finite: survives the bit packing
    wait_vmcnt<0>();
  }
  if (tid < ACC_MAXM) cnt_s[tid] = 0;
  int kaddr[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) kaddr[ks] = c * CROWB + (((ks * 2 + hb) ^ swz(c)) * 16);
  __syncthreads();

  // scores and arg-max, as assign_mfma
  float best[PB]; int btile[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) { best[pb] = -INFINITY; btile[pb] = 0; }
  for (int rb = 0; rb < CT; ++rb) {
    f32x16_t acc[PB];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float4 b4 = *reinterpret_cast<const float4*>(&bs[rb * 32 + 8 * i + 4 * hb]);
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) {
        acc[pb][4 * i + 0] = b4.x; acc[pb][4 * i + 1] = b4.y;
        acc[pb][4 * i + 2] = b4.z; acc[pb][4 * i + 3] = b4.w;
      }
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(pool + rb * 32 * CROWB + kaddr[ks]);
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) acc[pb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, xf[pb][ks], acc[pb], 0, 0, 0);
    }
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
      float pk[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) pk[v] = __uint_as_float((__float_as_uint(acc[pb][v]) & 0xFFFFFFF0u) | (uint32_t)(15 - v));
      float tm = fmaxf(fmaxf(pk[0], pk[1]), pk[2]);
#pragma unroll
      for (int v = 3; v < 15; v += 2) tm = fmaxf(fmaxf(tm, pk[v]), pk[v + 1]);
      tm = fmaxf(tm, pk[15]);
      if (tm > best[pb]) { best[pb] = tm; btile[pb] = rb; }
    }
  }
  int bidx[PB]; float bv[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
    const int v = 15 - (int)(__float_as_uint(best[pb]) & 15u);
    bidx[pb] = btile[pb] * 32 + 8 * (v >> 2) + 4 * hb + (v & 3);
    bv[pb] = __uint_as_float(__float_as_uint(best[pb]) & 0xFFFFFFF0u);
    const float ob = __shfl_xor(bv[pb], 32);
    const int oi = __shfl_xor(bidx[pb], 32);
    if (ob > bv[pb] || (ob == bv[pb] && oi < bidx[pb])) { bv[pb] = ob; bidx[pb] = oi; }
  }
  if (!out.psum) {
    // last pass: squared distances, and the survivors of the threshold or (first stage) the sum for it and the seeds of the
    // final pass
    int kept = 0;
    double dsum = 0.0;
    uint64_t keep[PB];
    const bool counts = cfg.keep_cnt != nullptr;
    const float t2 = counts ? cfg.tau[1] : 0.f;
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
      float ss = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const uint4 raw = *reinterpret_cast<const uint4*>(&xf[pb][ks]);
        const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float a = __uint_as_float(w[q] << 16), b = __uint_as_float(w[q] & 0xFFFF0000u);
          ss = fmaf(a, a, ss); ss = fmaf(b, b, ss);
        }
      }
      const float d2 = fmaxf(ss + __shfl_xor(ss, 32) - 2.f * bv[pb], 0.f);
      const bool mine = hb == 0 && pos[pb] < n;
      if (counts) {
        keep[pb] = __ballot(mine && !(d2 < t2));                         // (of the lower half-wave)
        kept += __popcll(keep[pb]);
      }
      if (mine) {
        dist2[(size_t)h * cfg.N + pos[pb]] = d2;
        if (cfg.dist_sum) dsum += (double)sqrtf(d2);
        if (cfg.keep_lab) { cfg.keep_lab[(size_t)h * cfg.N + pos[pb]] = bidx[pb]; cfg.keep_score[(size_t)h * cfg.N + pos[pb]] = bv[pb]; }
      }
    }
    __shared__ int32_t wkept[NW];
    __shared__ double wsum[NW];
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) dsum += __shfl_xor(dsum, o);      // (the upper half-wave holds zeros)
    if (lane == 0) { wkept[wave] = kept; wsum[wave] = dsum; }
    __syncthreads();
    if (tid == 0) {
      int k = 0; double s = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) { k += wkept[w]; s += wsum[w]; }
      if (counts) cfg.keep_cnt[(size_t)h * cfg.keep_stride + blockIdx.x] = k;
      if (cfg.dist_sum) cfg.dist_sum[(size_t)h * (gridDim.x - (FORM == PASS_OPEN ? 1 : 0)) + blockIdx.x] = s;
    }
    if (counts && cfg.surv && hb == 0) {   // the survivors in order, for the pass that opens the next stage
      int at = base;
      for (int w = 0; w < wave; ++w) at += wkept[w];
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) {
        if ((keep[pb] >> c) & 1) cfg.surv[(size_t)h * cfg.N + at + __popc((uint32_t)keep[pb] & ((1u << c) - 1u))] = tok[pb];
        else if (cfg.stage_of && pos[pb] < n) cfg.stage_of[(size_t)h * cfg.N + tok[pb]] = cfg.stage;
        at += __popcll(keep[pb]);
      }
    }
    return;
  }
  __syncthreads();                       // every wave is done with the centres: the points take their place
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
    const int pr = wave * (PB * 32) + pb * 32 + c;
    // Zeros for points past the last one: the row of a token that is not in this stage stands there, and zero times what is not finite
    // is NaN.  (Calls of 30 x 17 776, d=64, and 12 x 32 760, d=128, within 0.3 % of their time without.)
    if (FORM != PASS_OPEN && pos[pb] >= n) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) xf[pb][ks] = bf16x8_t{};
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) *reinterpret_cast<bf16x8_t*>(pool + pr * CROWB + (((ks * 2 + hb) ^ xswz(pr)) * 16)) = xf[pb][ks];
    if (hb == 0) {
      lab_s[pr] = pos[pb] < n ? bidx[pb] : -1;
      if (pos[pb] < n) atomicAdd(&cnt_s[bidx[pb]], 1);
    }
  }
  __syncthreads();
  // A wave takes a whole centre tile, so that the one-hot operand of a group of 16 points (twenty vector instructions,
  // more than the product it feeds) is built once and serves every dim tile; with fewer tiles than waves, R waves share
  // the points of a tile.
  const int b = blockIdx.x, R = m <= 32 ? NW : m <= 64 ? NW / 2 : NW / 4, G = 4 * NW / R, part = wave % R, ct = wave / R;
  const int i16 = lane & 15, blk = lane >> 4;
  const int vrow = 4 * hb + (i16 >> 2);
  const int gl = 2 * (blk & 1) + ((i16 & 3) >> 1);
  const int cid = ct * 32 + c;
  f32x16_t sacc[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) sacc[t][v] = 0.f;
  if (ct < CT) {
    // X^T operand by transpose reads (see the V operand of the attention kernel): this lane addresses
    // point 4*hb + (lane%16)/4 of a 16-point group, dims 16*((lane/16)%2) + 4*(lane%4) .. +3
    int xlo[DT], xhi[DT];
#pragma unroll
    for (int db = 0; db < DT; ++db) {
      xlo[db] = vrow * CROWB + (((db * 4 + gl) ^ xswz(vrow)) * 16) + 8 * (i16 & 1);
      xhi[db] = (vrow + 8) * CROWB + (((db * 4 + gl) ^ xswz(vrow + 8)) * 16) + 8 * (i16 & 1);
    }
#pragma unroll 4
    for (int g = part * G; g < part * G + G; ++g) {
      const int4 l0 = *reinterpret_cast<const int4*>(&lab_s[g * 16 + 4 * hb]);
      const int4 l1 = *reinterpret_cast<const int4*>(&lab_s[g * 16 + 8 + 4 * hb]);
      uint4 e;
      e.x = (l0.x == cid ? 0x3F80u : 0u) | (l0.y == cid ? 0x3F800000u : 0u);
      e.y = (l0.z == cid ? 0x3F80u : 0u) | (l0.w == cid ? 0x3F800000u : 0u);
      e.z = (l1.x == cid ? 0x3F80u : 0u) | (l1.y == cid ? 0x3F800000u : 0u);
      e.w = (l1.z == cid ? 0x3F80u : 0u) | (l1.w == cid ? 0x3F800000u : 0u);
      const bf16x8_t eb = *reinterpret_cast<const bf16x8_t*>(&e);
#pragma unroll
      for (int db = 0; db < DT; ++db) {
        const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(pool + g * 16 * CROWB + xlo[db]));
        const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(pool + g * 16 * CROWB + xhi[db]));
        const s16x4_t both[2] = {lo, hi};
        sacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8_t*>(both), eb, sacc[db], 0, 0, 0);
      }
    }
  }
  static_assert(NW * 32 * D * 4 <= NT * CROWB && ACC_MAXM == STAGE_COUNTS, "the partial sums fit the buffer of the points");
  store_sums<D, NW>(sacc, reinterpret_cast<float*>(pool), out, h, b, m, R, wave, c, hb);
  if (tid < m) out.bcnt[((size_t)h * out.nb_stride + b) * ACC_MAXM + tid] = cnt_s[tid];
}

// ------------------------------------------------------------------------------------------
// One pass of the query k-means in ONE read of the points: assignment and centroid sums together.
// ------------------------------------------------------------------------------------------
// A workgroup walks `subs` consecutive sub-blocks of 128 points.  Per sub-block every wave assigns its 32
// points to the nearest of the m <= 128 centres (all of them resident in LDS; the same MFMA product and in-lane
// arg-max as assign_mfma), then the sub-block's points, labels and weights go through LDS and every wave adds
//   S^T[32 dims x 32 centres] += X^T[32 dims x 16 points] . E[16 points x 32 centres]
// to the accumulator tiles it owns for the WHOLE walk (wave w: centre tile w in every dim tile).  E is the one-hot label matrix times the point's weight: 1 for Euclidean sums, and for the
// clustering by angle the bf16 value of 1/|x|, so that the tile holds the sum of the (almost) normalised
// members; the weight's rounding (2^-9 relative per member, of random sign) is far below the bf16 rounding the
// centres of the next assignment get anyway.  Products are exact, the accumulation is fp32 in a fixed order,
// so the pass is deterministic.  Walk b of head h leaves row j * NP + b of the head's part-sum table
// psum [H][m * NP][D] and pcnt[(h * NP + b) * ACC_MAXM + j]; finalize_centroids adds the walks in order.
// No label is written: only the last pass of a clustering needs labels, and that one takes the sorted path.
template <int D>
__global__ __launch_bounds__(256, 2) void qpass_mfma(const bf16raw* __restrict__ X, int N, int m, int cap, int subs,
                                                     int weighted, const bf16raw* __restrict__ cent,
                                                     const float* __restrict__ bias, float* __restrict__ psum,
                                                     int32_t* __restrict__ pcnt, int NP) {
  constexpr int KS = D / 16, DT = D / 32, ROWB = D * 2, CH = D / 8, SB = 128, MAXCT = ACC_MAXM / 32;
  const int h = blockIdx.y, b = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 31, hb = lane >> 5;
  const int CT = (m + 31) >> 5;
  __shared__ __attribute__((aligned(16))) char cs[MAXCT * 32 * ROWB];     // the centres, rows permuted by chunk
  __shared__ __attribute__((aligned(16))) float bs[MAXCT * 32];
  __shared__ __attribute__((aligned(16))) bf16raw xs[SB * D];             // the sub-block's points, row-major
  __shared__ __attribute__((aligned(16))) int32_t lab_s[SB];
  __shared__ __attribute__((aligned(16))) uint32_t w_s[SB];               // weight of a point as bf16 bits
  __shared__ int32_t cnt_s[ACC_MAXM];
  auto swz = [](int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); };
  {
    const bf16raw* chh = cent + (size_t)h * cap * D;
    for (int item = tid; item < CT * 32 * CH; item += 256) {
      const int r = item / CH, sl = item % CH;
      const int row = min(r, m - 1);                                      // rows past m repeat the last centre under a bias that never wins
      *reinterpret_cast<uint4*>(cs + r * ROWB + ((sl ^ swz(r)) * 16)) =
          *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(chh) + (size_t)row * ROWB + sl * 16);
    }
    if (tid < MAXCT * 32) { bs[tid] = tid < m ? bias[(size_t)h * cap + tid] : -3.0e38f; cnt_s[tid] = 0; }
  }
  int kaddr[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) kaddr[ks] = c * ROWB + (((ks * 2 + hb) ^ swz(c)) * 16);
  // Wave w owns centre tile w (there are at most four) in all its dim tiles: the one-hot operand of a group
  // of 16 points (about twenty vector instructions, more than one product costs) is built once per group
  // and serves every dim tile.
  f32x16_t sacc[DT];
#pragma unroll
  for (int k = 0; k < DT; ++k)
#pragma unroll
    for (int v = 0; v < 16; ++v) sacc[k][v] = 0.f;
  // X^T operand by transpose reads (as the V operand of the attention kernel): this lane addresses point
  // 4*hb + (lane%16)/4 of a 16-point group, dims 16*((lane/16)%2) + 4*(lane%4) .. +3
  const int i16 = lane & 15, blk = lane >> 4;
  const int vrow = 4 * hb + (i16 >> 2);
  const int gl = 2 * (blk & 1) + ((i16 & 3) >> 1);
  // Piece q (16 bytes) of point row r sits in slot q ^ xswz(r): a bijection over 16 consecutive rows (the
  // row-wise 16-byte writes of 16 lanes fall into 16 different bank groups) that also sends the four rows
  // of one transpose read to four different 64-byte groups.
  auto xswz = [](int r) { return D == 128 ? (((r & 3) << 2) | ((r >> 2) & 3)) : (((((r >> 1) & 7) & 1) << 2) | (((r >> 1) & 7) >> 1)); };
  int xlo[DT], xhi[DT];
#pragma unroll
  for (int db = 0; db < DT; ++db) {
    xlo[db] = vrow * ROWB + (((db * 4 + gl) ^ xswz(vrow)) * 16) + 8 * (i16 & 1);
    xhi[db] = (vrow + 8) * ROWB + (((db * 4 + gl) ^ xswz(vrow + 8)) * 16) + 8 * (i16 & 1);
  }
  const char* xsb = reinterpret_cast<const char*>(xs);

  const int p_begin = b * subs * SB;
  const bf16raw* Xh = X + (size_t)h * N * D;
  auto load_rows = [&](int base, bf16x8_t* xf) {
    const int pos = base + wave * 32 + c;
    if (pos < N) {
      const bf16raw* row = Xh + (size_t)pos * D + hb * 8;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) { const uint4 raw = *reinterpret_cast<const uint4*>(row + ks * 16); xf[ks] = *reinterpret_cast<const bf16x8_t*>(&raw); }
    } else {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) { const uint4 z = {0, 0, 0, 0}; xf[ks] = *reinterpret_cast<const bf16x8_t*>(&z); }
    }
  };
  bf16x8_t xnext[KS];
  load_rows(p_begin, xnext);
  __syncthreads();                       // centres, bias and counters are in LDS
  for (int sb = 0; sb < subs; ++sb) {
    const int base = p_begin + sb * SB;
    if (base >= N) break;
    bf16x8_t xf[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) xf[ks] = xnext[ks];
    if (sb + 1 < subs) load_rows(base + SB, xnext);          // the next sub-block's rows travel under this one's arithmetic
    const int pos = base + wave * 32 + c;
    // squared norm of this lane's point (both half-waves hold half of the row)
    float ss = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uint4 raw = *reinterpret_cast<const uint4*>(&xf[ks]);
      const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float a = __uint_as_float(w[q] << 16), bb = __uint_as_float(w[q] & 0xFFFF0000u);
        ss = fmaf(a, a, ss); ss = fmaf(bb, bb, ss);
      }
    }
    ss += __shfl_xor(ss, 32);
    // assignment: arg-max of x.c + bias over the centre tiles, position in a tile carried in the low 4 mantissa bits
    float best = -INFINITY; int btile = 0;
    for (int ct = 0; ct < CT; ++ct) {
      f32x16_t acc;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float4 b4 = *reinterpret_cast<const float4*>(&bs[ct * 32 + 8 * i + 4 * hb]);
        acc[4 * i + 0] = b4.x; acc[4 * i + 1] = b4.y; acc[4 * i + 2] = b4.z; acc[4 * i + 3] = b4.w;
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(cs + ct * 32 * ROWB + kaddr[ks]);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, xf[ks], acc, 0, 0, 0);
      }
      float pk[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) pk[v] = __uint_as_float((__float_as_uint(acc[v]) & 0xFFFFFFF0u) | (uint32_t)(15 - v));
      float tm = fmaxf(fmaxf(pk[0], pk[1]), pk[2]);
#pragma unroll
      for (int v = 3; v < 15; v += 2) tm = fmaxf(fmaxf(tm, pk[v]), pk[v + 1]);
      tm = fmaxf(tm, pk[15]);
      if (tm > best) { best = tm; btile = ct; }
    }
    {
      const int v = 15 - (int)(__float_as_uint(best) & 15u);
      int bidx = btile * 32 + 8 * (v >> 2) + 4 * hb + (v & 3);
      float bv = __uint_as_float(__float_as_uint(best) & 0xFFFFFFF0u);
      const float ob = __shfl_xor(bv, 32);
      const int oi = __shfl_xor(bidx, 32);
      if (ob > bv || (ob == bv && oi < bidx)) { bv = ob; bidx = oi; }
      const int pr = wave * 32 + c;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        *reinterpret_cast<bf16x8_t*>(reinterpret_cast<char*>(xs) + pr * ROWB + (((ks * 2 + hb) ^ xswz(pr)) * 16)) = xf[ks];
      if (hb == 0) {
        const bool valid = pos < N;
        lab_s[pr] = valid ? bidx : -1;
        w_s[pr] = weighted ? (uint32_t)f32_to_bf16(1.0f / fmaxf(sqrtf(ss), 1e-12f)) : 0x3F80u;
        if (valid) atomicAdd(&cnt_s[bidx], 1);
      }
    }
    __syncthreads();
    // sums: the owned centre tile takes the eight 16-point groups of the sub-block
    if (wave < CT) {
      const int cid = wave * 32 + c;
#pragma unroll 2
      for (int g = 0; g < SB / 16; ++g) {
        const int4 l0 = *reinterpret_cast<const int4*>(&lab_s[g * 16 + 4 * hb]);
        const int4 l1 = *reinterpret_cast<const int4*>(&lab_s[g * 16 + 8 + 4 * hb]);
        const uint4 w0 = *reinterpret_cast<const uint4*>(&w_s[g * 16 + 4 * hb]);
        const uint4 w1 = *reinterpret_cast<const uint4*>(&w_s[g * 16 + 8 + 4 * hb]);
        uint4 e;
        e.x = (l0.x == cid ? w0.x : 0u) | (l0.y == cid ? w0.y << 16 : 0u);
        e.y = (l0.z == cid ? w0.z : 0u) | (l0.w == cid ? w0.w << 16 : 0u);
        e.z = (l1.x == cid ? w1.x : 0u) | (l1.y == cid ? w1.y << 16 : 0u);
        e.w = (l1.z == cid ? w1.z : 0u) | (l1.w == cid ? w1.w << 16 : 0u);
        const bf16x8_t eb = *reinterpret_cast<const bf16x8_t*>(&e);
#pragma unroll
        for (int db = 0; db < DT; ++db) {
          const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(xsb + g * 16 * ROWB + xlo[db]));
          const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(xsb + g * 16 * ROWB + xhi[db]));
          const s16x4_t both[2] = {lo, hi};
          sacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8_t*>(both), eb, sacc[db], 0, 0, 0);
        }
      }
    }
    __syncthreads();                     // the sub-block's points and labels may be overwritten
  }
  // value v of dim tile db is dim db*32 + 8*(v/4) + 4*hb + v%4 of centre cid
  if (wave < CT && wave * 32 + c < m) {
    const int cid = wave * 32 + c;
#pragma unroll
    for (int db = 0; db < DT; ++db) {
      float* out = psum + ((size_t)h * m * NP + (size_t)cid * NP + b) * D + db * 32 + 4 * hb;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float4 o4 = {sacc[db][4 * i], sacc[db][4 * i + 1], sacc[db][4 * i + 2], sacc[db][4 * i + 3]};
        *reinterpret_cast<float4*>(out + 8 * i) = o4;
      }
    }
  }
  if (tid < m) pcnt[((size_t)h * NP + b) * ACC_MAXM + tid] = cnt_s[tid];
}

// fp32 I/O: the same product with v_mfma_f32_32x32x2_f32.  A chain of these is, to the bit, the chain of fused multiply-adds
// in ascending dimension order (step s contracts the dims 2s, from the lower half-wave, and 2s + 1, from the upper one), so
// scores, labels and distances are those of a thread that takes its point's products one after the other.
// A workgroup is 64 points, two groups of 32, and 128 centres at a time in LDS, a tile of 32 for each of four waves of either
// group; the four meet at the end.  What bounds it is how few waves such calls have: the fp32 matrix rate is the vector rate,
// but a wave here is 32 points x a quarter of the centres; with a point a thread against all of them (3 x 5 007 points: a
// quarter of the SIMDs had a wave), an LDS read for every four multiply-adds, it was 47 us with 65 centres, d=128, and 184
// with 288, now 11 and 19; 4 x 12 000 points, 100 centres 72 -> 25; 4 096, d=64, 32 centres 15 -> 5; 24 x 20 000, d=128, 65
// and 1 024 centres 219 -> 184 and 2 690 -> 1 070 (118 TFLOP/s).  With rows straight into registers, every wave its own
// copy, 16 instead of 11 us, and 381 instead of 184 in the large launch; 128 registers and two workgroups a CU: 239 -> 184.
// Piece q (16 bytes) of centre row r sits in slot q ^ (r & 15) of its 256 bytes: a read of 32 rows meets every bank twice.
// NS = 1, with at most 32 centres: one tile, and its two waves are the workgroup (30 x 3 000 points, 8 centres: the other six
// waves of 1 400 workgroups made a pass 20 us instead of 14).  Few centres in large launches go to assign_rows.
template <int D, int NS>
__global__ __launch_bounds__(NS * 64 * (ASSIGN_POINTS_F32 / 32), 4) void assign_f32(const float* __restrict__ X, AssignCfg cfg,
                                                  const float* __restrict__ cent,
                                                  const float* __restrict__ bias,
                                                  int32_t* __restrict__ labels, float* __restrict__ dist2) {
  constexpr int PG = ASSIGN_POINTS_F32 / 32, CB = 32 * NS, ROWB = D * 4, PPR = D / 4, NT = 64 * NS * PG;
  constexpr int ROWS = CB > ASSIGN_POINTS_F32 + 32 ? CB : ASSIGN_POINTS_F32 + 32;      // of LDS
  const int h = blockIdx.y;
  int n, m, row_off;
  if (!assign_setup(cfg, h, n, m, row_off)) return;
  const int base = blockIdx.x * ASSIGN_POINTS_F32;
  if (base >= n) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 31, hb = lane >> 5, pg = wave % PG, sp = wave / PG;     // (waves of the first tile on different SIMDs)
  __shared__ __attribute__((aligned(16))) char cs[ROWS * ROWB];
  __shared__ __attribute__((aligned(16))) float bs[CB];
  __shared__ float sbest[NS][ASSIGN_POINTS_F32];
  __shared__ int32_t sidx[NS][ASSIGN_POINTS_F32];
  const char* ch = reinterpret_cast<const char*>(cent + ((size_t)h * cfg.cap + row_off) * D);
  const float* bh = bias + (size_t)h * cfg.cap + row_off;
  const uint32_t cs0 = (uint32_t)(uintptr_t)(lds_void_t*)cs;
  auto issue_chunk = [&](int c0) __attribute__((always_inline)) {       // whole tiles; rows past m repeat the last centre
    const int rows = min(CB, (m - c0 + 31) & ~31);
#pragma unroll
    for (int i = 0; i < CB * PPR / NT; ++i) {
      const int item = tid + i * NT, r = item / PPR, sl = item % PPR, q = (sl & ~15) | ((sl ^ r) & 15);
      if (r < rows) dma_b128(cs0 + (wave * 64 + i * NT) * 16, ch + (size_t)min(c0 + r, m - 1) * ROWB + q * 16);
    }
    for (int i = tid; i < CB; i += NT) bs[i] = c0 + i < m ? bh[c0 + i] : -INFINITY;
  };
  // The points come through LDS: beside the first chunk of centres where that leaves room, else before it.
  const bool beside = m <= ROWS - ASSIGN_POINTS_F32;
  char* const ps = cs + (beside ? (ROWS - ASSIGN_POINTS_F32) * ROWB : 0);
#pragma unroll
  for (int i = 0; i < ASSIGN_POINTS_F32 * PPR / NT; ++i) {
    const int item = tid + i * NT, r = item / PPR, sl = item % PPR, q = (sl & ~15) | ((sl ^ r) & 15);
    const int pr = min(base + r, n - 1), tok = cfg.ulist ? cfg.ulist[(size_t)h * cfg.N + pr] : pr;
    dma_b128((uint32_t)(uintptr_t)(lds_void_t*)ps + (wave * 64 + i * NT) * 16, reinterpret_cast<const char*>(X + ((size_t)h * cfg.N + tok) * D) + q * 16);
  }
  if (beside && m > 0) issue_chunk(0);
  const int p = base + pg * 32 + c;
  float x[D / 2], xn2 = 0.f;            // this half-wave's dims: 2s + hb
  wait_vmcnt<0>();
  __syncthreads();
  {
    const char* row = ps + (pg * 32 + c) * ROWB;
    const int sw = (c & 15) * 16;
#pragma unroll
    for (int q = 0; q < PPR; ++q) {
      const float* a = reinterpret_cast<const float*>(row + ((((q & 15) * 16) ^ sw) + (q >> 4) * 256) + hb * 4);
      x[2 * q] = a[0]; x[2 * q + 1] = a[2];
    }
    if (dist2 && sp == 0) {
#pragma unroll 8
      for (int q = 0; q < PPR; ++q) {
        const float4 v = *reinterpret_cast<const float4*>(row + ((((q & 15) * 16) ^ sw) + (q >> 4) * 256));
        xn2 = fmaf(v.x, v.x, xn2); xn2 = fmaf(v.y, v.y, xn2); xn2 = fmaf(v.z, v.z, xn2); xn2 = fmaf(v.w, v.w, xn2);
      }
    }
  }
  if (!beside) {
    __syncthreads();
    issue_chunk(0);
  }
  float best = -INFINITY; int bidx = 0;
  for (int c0 = 0; c0 < m; c0 += CB) {
    wait_vmcnt<0>();                    // this wave's pieces of the chunk are in LDS
    __syncthreads();
    const int j0 = c0 + sp * 32;
    if (j0 < m) {
      f32x16_t acc;
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[v] = 0.f;
      const char* tile = cs + sp * 32 * ROWB;
      const int a0 = c * ROWB + ((c & 15) * 16) + hb * 4;
      auto piece = [&](int q) __attribute__((always_inline)) {       // dims 4q + hb and 4q + 2 + hb of row c
        const float* a = reinterpret_cast<const float*>(tile + ((a0 ^ ((q & 15) * 16)) + (q >> 4) * 256));
        return float2{a[0], a[2]};
      };
      constexpr int AHEAD = 4;
      float2 kb[AHEAD];
#pragma unroll
      for (int q = 0; q < AHEAD; ++q) kb[q] = piece(q);
#pragma unroll
      for (int q = 0; q < PPR; ++q) {
        const float2 a = kb[q % AHEAD];
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, x[2 * q], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, x[2 * q + 1], acc, 0, 0, 0);
        if (q + AHEAD < PPR) kb[q % AHEAD] = piece(q + AHEAD);
      }
      // value v is centre j0 + 8*(v/4) + 4*hb + v%4: ascending in v
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int jr = 8 * (v >> 2) + 4 * hb + (v & 3);
        const float s = acc[v] + bs[sp * 32 + jr];
        if (s > best) { best = s; bidx = j0 + jr; }
      }
    }
    if (c0 + CB < m) {
      __syncthreads();                  // every wave is done with the chunk
      issue_chunk(c0 + CB);
    }
  }
  {
    const float ob = __shfl_xor(best, 32);
    const int oi = __shfl_xor(bidx, 32);
    if (ob > best || (ob == best && oi < bidx)) { best = ob; bidx = oi; }
  }
  if (hb == 0) { sbest[sp][pg * 32 + c] = best; sidx[sp][pg * 32 + c] = bidx; }
  __syncthreads();
  const bool mine = sp == 0 && hb == 0 && p < n;
  float d2 = 0.f;
  if (mine) {
#pragma unroll
    for (int w = 1; w < NS; ++w) {
      const float ob = sbest[w][pg * 32 + c];
      const int oi = sidx[w][pg * 32 + c];
      if (ob > best || (ob == best && oi < bidx)) { best = ob; bidx = oi; }
    }
    d2 = fmaxf(xn2 - 2.f * best, 0.f);
    labels[(size_t)h * cfg.N + p] = bidx;
    if (dist2) dist2[(size_t)h * cfg.N + p] = d2;
  }
  if (cfg.keep_cnt && dist2) {
    __shared__ int32_t wkept[PG];
    const uint64_t kept = __ballot(mine && !(d2 < cfg.tau[1]));
    if (sp == 0 && lane == 0) wkept[pg] = __popcll(kept);
    __syncthreads();
    if (tid == 0) cfg.keep_cnt[(size_t)h * cfg.keep_stride + blockIdx.x] = wkept[0] + wkept[1];
  }
  if (cfg.dist_sum) {
    double dsum = mine ? (double)sqrtf(d2) : 0.0;
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) dsum += __shfl_xor(dsum, o);      // (the upper half-wave holds zeros)
    __shared__ double wsum[PG];
    if (sp == 0 && lane == 0) wsum[pg] = dsum;
    __syncthreads();
    if (tid == 0) cfg.dist_sum[(size_t)h * gridDim.x + blockIdx.x] = wsum[0] + wsum[1];
  }
}

// ------------------------------------------------------------------------------------------
// A pass of a stage of Algorithm 1 with at most PASS_F32_CENTRES centres, fp32: what stage_pass is for bf16
// ------------------------------------------------------------------------------------------
// A workgroup is a block of PASS_F32_POINTS points in four groups of 32, eight waves: a group and one of two tiles of 32 centres each.
// Scores and labels are those of assign_f32, to the bit.  An update pass then leaves the members' sums: a wave takes every eighth
// centre, finds its members by two ballots over the labels, and adds their rows out of LDS, a lane a column.  Sums are formed in
// fp64, by blocks and then over the blocks (block_mean_f32), and rounded once, by the mean: the same members give the same centre
// in every stage, wherever in U they are (as in update_direct_f32, whose order does not depend on that), so that such centres tie
// exactly.  A call therefore takes the one or the other for all of its stages, and by its width, tokens and centres alone, so that a
// head has the same bits among any number of others.  (fp64 sums there as well: 6 000 points, d=64, 25 -> 43 us a launch.)
// Latency bound in small launches, 7-10 us: it takes the place of an assignment (5) and half of an update by label scan (5-7), and
// opens its stage (stage_open, 6-7).  In large ones a CU holds three workgroups, at d=128 one (102 KB of LDS).
// The blocks of a head start at another workgroup than those of the head before: workgroups go to the XCDs in turn, and where the
// blocks of a head are a multiple of eight, the first ones, which late stages have left, would all be on the first XCDs (24 x 4 000
// points, d=128, 360 -> 320 us a key clustering, 60 x 4 000 699 -> 616).
constexpr int PASS_F32_POINTS = 128, PASS_F32_CENTRES = 64;
// Mean of the members of centre j, columns 4 cl .. 4 cl + 3, from the sums of the blocks in their order, and the number of members (0: no
// mean).  By the D / 4 lanes of a centre together.
template <int D>
__device__ __forceinline__ float4 block_mean_f32(const PassSums& sums, int h, int j, int nb, int cl, int& nj) {
  constexpr int LPC = D / 4, BATCH = D == 64 ? 8 : 16;
  nj = 0;
  for (int b = cl; b < nb; b += LPC) nj += sums.bcnt[((size_t)h * sums.nb_stride + b) * STAGE_COUNTS + j];
  const double2* row = reinterpret_cast<const double2*>(reinterpret_cast<const double*>(sums.psum) + ((size_t)h * sums.P + (size_t)j * sums.nb_stride) * D + cl * 4);
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
  for (int b0 = 0; b0 < nb; b0 += BATCH) {
    double2 t[BATCH][2];
#pragma unroll
    for (int u = 0; u < BATCH; ++u) { const size_t o = (size_t)min(b0 + u, nb - 1) * (D / 2); t[u][0] = row[o]; t[u][1] = row[o + 1]; }
#pragma unroll
    for (int u = 0; u < BATCH; ++u) if (b0 + u < nb) { s0 += t[u][0].x; s1 += t[u][0].y; s2 += t[u][1].x; s3 += t[u][1].y; }
  }
#pragma unroll
  for (int o = 1; o < LPC; o <<= 1) nj += __shfl_xor(nj, o);
  const double cnt = (double)nj;
  return float4{(float)(s0 / cnt), (float)(s1 / cnt), (float)(s2 / cnt), (float)(s3 / cnt)};
}
// ... and the bias of centre r in the arg-max, -|r|^2 / 2.
template <int D>
__device__ __forceinline__ float centre_bias_f32(const float4& r) {
  float ss = fmaf(r.x, r.x, 0.f);
  ss = fmaf(r.y, r.y, ss); ss = fmaf(r.z, r.z, ss); ss = fmaf(r.w, r.w, ss);
#pragma unroll
  for (int o = 1; o < D / 4; o <<= 1) ss += __shfl_xor(ss, o);
  return -0.5f * ss;
}
template <int D, int FORM>
__global__ __launch_bounds__(512, D == 128 ? 2 : FORM == PASS_COMBINE ? 4 : 6) void stage_pass_f32(const float* __restrict__ X, AssignCfg cfg, float* __restrict__ cent,
                                                                       float* __restrict__ cent_f32, float* __restrict__ bias,
                                                                       float* __restrict__ dist2, int nblk, uint32_t turns, PassSums prev, PassSums out, OpenCfg oc) {
  constexpr bool OPEN = FORM == PASS_OPEN;
  constexpr int NT = 512, NP = PASS_F32_POINTS, MAXM = PASS_F32_CENTRES, ROWB = D * 4, PPR = D / 4, CPL = D / 64;
  const int h = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 31, hb = lane >> 5, pg = wave & 3, sp = wave >> 2;
  int n, m, row_off, t = 0;
  __shared__ int32_t pre[OPEN ? OPEN_COUNTS + 1 : 1], ctok[OPEN ? MAXM : 1];
  int b = blockIdx.x;
  if (FORM != PASS_COMBINE && nblk > 1) {                 // (small launches need no turn)
    b += h - (int)__umulhi((uint32_t)h, turns) * nblk;    // h % nblk, of at most 2^16 heads and 2^7 blocks
    if (b >= nblk) b -= nblk;
  }
  const int base = b * NP;
  if constexpr (OPEN) {
    if (!open_stage(oc, h, pre, n, m, row_off)) return;
  } else {
    if (tid < NP && cfg.ulist) t = cfg.ulist[(size_t)h * cfg.N + min(base + tid, cfg.N - 1)];      // (with the state, as in stage_pass)
    if (!assign_setup(cfg, h, n, m, row_off)) return;
  }
  if (base >= n) return;
  m = min(m, MAXM);
  const int CT = (m + 31) >> 5;
  __shared__ __attribute__((aligned(16))) char ps[NP * ROWB];
  __shared__ __attribute__((aligned(16))) char cs[MAXM * ROWB];
  __shared__ __attribute__((aligned(16))) float bs[MAXM];
  __shared__ float sbest[2][NP];
  __shared__ int32_t sidx[2][NP], tok_s[NP], lab_s[NP];
  const float* Xh = X + (size_t)h * cfg.N * D;
  auto slot_of = [](int r, int q) { return (q & ~15) | ((q ^ r) & 15); };       // where piece q (16 bytes) of row r is, as in assign_f32
  // tokens of the points (one of any for those past the last), and (opening) of the centres, survivor floor((2j+1) n / 2m)
  if (OPEN && tid < NP + MAXM) {
    const bool point = tid < NP;
    int at[1] = {point ? min(base + tid, n - 1) : sample_at(min(tid - NP, m - 1), n, m)};
    if (!oc.first) {
      survivors_at(pre, oc.items, at);
      at[0] = oc.surv[(size_t)h * cfg.N + at[0]];
      if (point && base + tid < n) oc.uout[(size_t)h * cfg.N + base + tid] = at[0];
    }
    if (point) tok_s[tid] = at[0];
    else if (tid - NP < m) ctok[tid - NP] = at[0];
  } else if (!OPEN && tid < NP) {
    tok_s[tid] = base + tid >= n ? 0 : cfg.ulist ? t : base + tid;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NP * PPR / NT; ++i) {
    const int item = tid + i * NT, r = item / PPR;
    dma_b128((uint32_t)(uintptr_t)(lds_void_t*)ps + (wave * 64 + i * NT) * 16, reinterpret_cast<const char*>(Xh + (size_t)tok_s[r] * D) + slot_of(r, item % PPR) * 16);
  }
  const size_t crow = (size_t)h * cfg.cap + row_off;
  if constexpr (FORM == PASS_READ) {
#pragma unroll
    for (int i = 0; i < MAXM * PPR / NT; ++i) {           // whole tiles; rows past m repeat the last centre
      const int item = tid + i * NT, r = item / PPR;
      if (r < CT * 32)
        dma_b128((uint32_t)(uintptr_t)(lds_void_t*)cs + (wave * 64 + i * NT) * 16, reinterpret_cast<const char*>(cent + (crow + min(r, m - 1)) * D) + slot_of(r, item % PPR) * 16);
    }
    if (tid < CT * 32) bs[tid] = tid < m ? bias[crow + tid] : -INFINITY;
  } else {
    const int cl = tid % PPR, nb = (n + NP - 1) / NP;
    for (int j = tid / PPR; j < CT * 32; j += NT / PPR) {
      float4 r = {0.f, 0.f, 0.f, 0.f};
      float bj = -INFINITY;
      if (j < m) {
        const size_t at = (crow + j) * D + cl * 4;
        int nj = 1;
        if constexpr (FORM == PASS_COMBINE) r = block_mean_f32<D>(prev, h, j, nb, cl, nj);
        else r = *reinterpret_cast<const float4*>(Xh + (size_t)ctok[j] * D + cl * 4);
        if (nj > 0) {
          bj = centre_bias_f32<D>(r);
          if (b == 0) {
            *reinterpret_cast<float4*>(cent + at) = r;
            *reinterpret_cast<float4*>(cent_f32 + at) = r;
            if (cl == 0) bias[crow + j] = bj;
          }
        } else {                                         // an empty cluster keeps its centre
          r = *reinterpret_cast<const float4*>(cent + at);
          bj = bias[crow + j];
        }
      }
      *reinterpret_cast<float4*>(cs + j * ROWB + slot_of(j, cl) * 16) = r;
      if (cl == 0) bs[j] = bj;
    }
  }
  wait_vmcnt<0>();
  __syncthreads();

  // scores and arg-max, as assign_f32
  const int p = base + pg * 32 + c;
  float best = -INFINITY, xn2 = 0.f;
  int bidx = 0;
  {
    float x[D / 2];                       // this half-wave's dims: 2s + hb
    const char* row = ps + (pg * 32 + c) * ROWB;
#pragma unroll
    for (int q = 0; q < PPR; ++q) {
      const float* a = reinterpret_cast<const float*>(row + slot_of(c, q) * 16 + hb * 4);
      x[2 * q] = a[0]; x[2 * q + 1] = a[2];
    }
    if (!out.psum && sp == 0) {
#pragma unroll 8
      for (int q = 0; q < PPR; ++q) {
        const float4 v = *reinterpret_cast<const float4*>(row + slot_of(c, q) * 16);
        xn2 = fmaf(v.x, v.x, xn2); xn2 = fmaf(v.y, v.y, xn2); xn2 = fmaf(v.z, v.z, xn2); xn2 = fmaf(v.w, v.w, xn2);
      }
    }
    if (sp < CT) {
      f32x16_t acc;
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[v] = 0.f;
      const char* tile = cs + (sp * 32 + c) * ROWB + hb * 4;
#pragma unroll
      for (int q = 0; q < PPR; ++q) {
        const float* a = reinterpret_cast<const float*>(tile + slot_of(c, q) * 16);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[0], x[2 * q], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[2], x[2 * q + 1], acc, 0, 0, 0);
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int j = sp * 32 + 8 * (v >> 2) + 4 * hb + (v & 3);
        const float s = acc[v] + bs[j];
        if (s > best) { best = s; bidx = j; }
      }
    }
  }
  {
    const float ob = __shfl_xor(best, 32);
    const int oi = __shfl_xor(bidx, 32);
    if (ob > best || (ob == best && oi < bidx)) { best = ob; bidx = oi; }
  }
  if (hb == 0) { sbest[sp][pg * 32 + c] = best; sidx[sp][pg * 32 + c] = bidx; }
  __syncthreads();
  const bool mine = sp == 0 && hb == 0 && p < n;
  if (mine) {
    const float ob = sbest[1][pg * 32 + c];
    const int oi = sidx[1][pg * 32 + c];
    if (ob > best || (ob == best && oi < bidx)) { best = ob; bidx = oi; }
  }
  if (!out.psum) {
    // last pass: squared distances, and the survivors of the threshold or (first stage) the sum for it
    const float d2 = fmaxf(xn2 - 2.f * best, 0.f);
    const bool counts = cfg.keep_cnt != nullptr;
    const uint64_t keep = __ballot(mine && counts && !(d2 < cfg.tau[1]));
    double dsum = mine && cfg.dist_sum ? (double)sqrtf(d2) : 0.0;
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) dsum += __shfl_xor(dsum, o);      // (the upper half-wave holds zeros)
    __shared__ int32_t wkept[4];
    __shared__ double wsum[4];
    if (sp == 0 && lane == 0) { wkept[pg] = __popcll(keep); wsum[pg] = dsum; }
    if (mine) dist2[(size_t)h * cfg.N + p] = d2;
    __syncthreads();
    if (tid == 0) {
      if (counts) cfg.keep_cnt[(size_t)h * cfg.keep_stride + b] = (wkept[0] + wkept[1]) + (wkept[2] + wkept[3]);
      if (cfg.dist_sum) cfg.dist_sum[(size_t)h * nblk + b] = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
    }
    if (counts && cfg.surv && mine) {      // the survivors in order, for the pass that opens the next stage
      int at = base;
      for (int w = 0; w < pg; ++w) at += wkept[w];
      const int t = tok_s[pg * 32 + c];
      if ((keep >> c) & 1) cfg.surv[(size_t)h * cfg.N + at + __popc((uint32_t)keep & ((1u << c) - 1u))] = t;
      else if (cfg.stage_of) cfg.stage_of[(size_t)h * cfg.N + t] = cfg.stage;
    }
    return;
  }
  if (sp == 0 && hb == 0) lab_s[pg * 32 + c] = mine ? bidx : -1;
  __syncthreads();
  const int l0 = lab_s[lane], l1 = lab_s[64 + lane];
  auto value = [&](int r, int q) { const int col = lane + 64 * q; return *reinterpret_cast<const float*>(ps + r * ROWB + slot_of(r, col >> 2) * 16 + (col & 3) * 4); };
  for (int j = wave; j < m; j += 8) {
    uint64_t left[2] = {__ballot(l0 == j), __ballot(l1 == j)};
    double sum[CPL];
#pragma unroll
    for (int q = 0; q < CPL; ++q) sum[q] = 0.0;
    const int members = __popcll(left[0]) + __popcll(left[1]);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      while (left[half]) {                // four members at a time, in their order
        float v[4][CPL];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const bool in = left[half] != 0;
          const int r = 64 * half + (in ? __ffsll((unsigned long long)left[half]) - 1 : 0);
          left[half] &= left[half] - 1;
#pragma unroll
          for (int q = 0; q < CPL; ++q) { const float x = value(r, q); v[u][q] = in ? x : 0.f; }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int q = 0; q < CPL; ++q) sum[q] += (double)v[u][q];
      }
    }
    double* row = reinterpret_cast<double*>(out.psum) + ((size_t)h * out.P + (size_t)j * out.nb_stride + b) * D;
#pragma unroll
    for (int q = 0; q < CPL; ++q) row[lane + 64 * q] = sum[q];
    if (lane == 0) out.bcnt[((size_t)h * out.nb_stride + b) * STAGE_COUNTS + j] = members;
  }
}

// The centres of a stage from the sums that stage_pass_f32 left, in a launch of their own: what PASS_COMBINE makes of them, to the bit
// (pass_f32_combines() says when).
template <int D>
__global__ __launch_bounds__(256) void form_centres_f32(PassSums sums, const KState* __restrict__ st, int cap, float* __restrict__ cent,
                                                        float* __restrict__ cent_f32, float* __restrict__ bias) {
  constexpr int LPC = D / 4;
  const int h = blockIdx.y, j = blockIdx.x * (256 / LPC) + threadIdx.x / LPC, cl = threadIdx.x % LPC;
  const KState& s = st[h];
  if (!s.active || j >= min(s.m_t, PASS_F32_CENTRES)) return;
  int nj;
  const float4 r = block_mean_f32<D>(sums, h, j, (s.ucount + PASS_F32_POINTS - 1) / PASS_F32_POINTS, cl, nj);
  if (nj == 0) return;                   // an empty cluster keeps its centre
  const float bj = centre_bias_f32<D>(r);
  const size_t row = (size_t)h * cap + s.ccount + j;
  *reinterpret_cast<float4*>(cent + row * D + cl * 4) = r;
  *reinterpret_cast<float4*>(cent_f32 + row * D + cl * 4) = r;
  if (cl == 0) bias[row] = bj;
}

// The same scores, labels, distances and counts, to the bit, from a point a thread and centres broadcast from LDS: vector
// multiply-adds for the centres that there are, where assign_f32 takes whole tiles of 32 and its points twice through LDS.
// assign_f32_rows() says when.
constexpr int ROWS_POINTS = 128;
static_assert(ROWS_POINTS == 2 * ASSIGN_POINTS_F32 && ASSIGN_POINTS_F32 == 64, "a wave's points are those of a count");
template <int D>
__global__ __launch_bounds__(ROWS_POINTS) void assign_rows(const float* __restrict__ X, AssignCfg cfg,
                                                           const float* __restrict__ cent,
                                                           const float* __restrict__ bias,
                                                           int32_t* __restrict__ labels, float* __restrict__ dist2) {
  constexpr int CB = 32;
  const int h = blockIdx.y;
  int n, m, row_off;
  if (!assign_setup(cfg, h, n, m, row_off)) return;
  const int base = blockIdx.x * ROWS_POINTS;
  if (base >= n) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int p = base + tid;
  __shared__ __attribute__((aligned(16))) float cs[CB * D];
  __shared__ float bs[CB];
  float x[D];
  float xn2 = 0.f;
  if (p < n) {
    const int tok = cfg.ulist ? cfg.ulist[(size_t)h * cfg.N + p] : p;
    const float4* row = reinterpret_cast<const float4*>(X + ((size_t)h * cfg.N + tok) * D);
#pragma unroll
    for (int q = 0; q < D / 4; ++q) {
      const float4 v = row[q];
      x[4 * q] = v.x; x[4 * q + 1] = v.y; x[4 * q + 2] = v.z; x[4 * q + 3] = v.w;
    }
#pragma unroll
    for (int j = 0; j < D; ++j) xn2 = fmaf(x[j], x[j], xn2);
  } else {
#pragma unroll
    for (int j = 0; j < D; ++j) x[j] = 0.f;
  }
  const float* ch = cent + ((size_t)h * cfg.cap + row_off) * D;
  const float* bh = bias + (size_t)h * cfg.cap + row_off;
  float best = -INFINITY; int bidx = 0;
  for (int c0 = 0; c0 < m; c0 += CB) {
    __syncthreads();
    for (int i = tid; i < CB * D / 4; i += ROWS_POINTS) {
      const int r = i / (D / 4);
      float4 v = {0.f, 0.f, 0.f, 0.f};
      if (c0 + r < m) v = reinterpret_cast<const float4*>(ch + (size_t)c0 * D)[i];
      reinterpret_cast<float4*>(cs)[i] = v;
    }
    if (tid < CB) bs[tid] = (c0 + tid < m) ? bh[c0 + tid] : -INFINITY;
    __syncthreads();
    const int rmax = min(CB, m - c0);
    for (int r = 0; r < rmax; ++r) {
      float s = 0.f;
#pragma unroll
      for (int q = 0; q < D / 4; ++q) {
        const float4 v = *reinterpret_cast<const float4*>(&cs[r * D + 4 * q]);
        s = fmaf(x[4 * q], v.x, s); s = fmaf(x[4 * q + 1], v.y, s);
        s = fmaf(x[4 * q + 2], v.z, s); s = fmaf(x[4 * q + 3], v.w, s);
      }
      s += bs[r];
      if (s > best) { best = s; bidx = c0 + r; }
    }
  }
  const float d2 = fmaxf(xn2 - 2.f * best, 0.f);
  if (p < n) {
    labels[(size_t)h * cfg.N + p] = bidx;
    if (dist2) dist2[(size_t)h * cfg.N + p] = d2;
  }
  // a wave's 64 points are a workgroup of assign_f32 (the last workgroup may have none for its second wave)
  const int part = 2 * blockIdx.x + wave;
  const bool any = base + wave * 64 < n;
  if (cfg.keep_cnt && dist2) {
    const uint64_t kept = __ballot(p < n && !(d2 < cfg.tau[1]));
    if (any && lane == 0) cfg.keep_cnt[(size_t)h * cfg.keep_stride + part] = __popcll(kept);
  }
  if (cfg.dist_sum) {                                    // (over all points: the first stage)
    double dsum = p < n ? (double)sqrtf(d2) : 0.0;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) dsum += __shfl_xor(dsum, o);
    if (any && lane == 0) cfg.dist_sum[(size_t)h * ((cfg.N + 63) / 64) + part] = dsum;
  }
}

// ------------------------------------------------------------------------------------------
// centroid update: segmented sums over the sorted order (no atomics, fixed summation order)
// ------------------------------------------------------------------------------------------
struct ReduceCfg {
  int mode;            // same meaning as AssignCfg::mode (where m and activity come from)
  int m_const; int N; int P /* upper bound of parts per head = grid.x */; int m_bound;
  const KState* st;
  int normalize;       // rows are scaled to unit length before summing (query clustering)
  int want_box;
};

__device__ __forceinline__ bool reduce_setup(const ReduceCfg& c, int h, int& m) {
  if (c.mode == 0) { m = c.m_const; return true; }
  const KState& s = c.st[h];
  if (c.mode == 1) { m = s.m_t; return s.active != 0; }
  m = s.ccount; return true;
}

// One wave sums one part of one cluster with 16-byte loads: a row is covered by LPR lanes, the
// wave takes RPI = 64/LPR rows per step (two steps in flight), and the RPI row slots are merged
// at the end in a fixed order, so the result does not depend on scheduling.
// psum [H][m_bound][P][D]; pnorm [H][m_bound][P]; pmin/pmax like psum.
static constexpr int REDUCE_ROWS = 128;   // rows summed by one wave (64, 96 and 192 measured the same)

template <typename T> struct Vec16;
template <> struct Vec16<bf16raw> {
  static constexpr int N = 8;
  static __device__ __forceinline__ void decode(const uint4 r, float* x) {
    const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) { x[2 * i] = __uint_as_float(w[i] << 16); x[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u); }
  }
};
template <> struct Vec16<float> {
  static constexpr int N = 4;
  static __device__ __forceinline__ void decode(const uint4 r, float* x) {
    x[0] = __uint_as_float(r.x); x[1] = __uint_as_float(r.y); x[2] = __uint_as_float(r.z); x[3] = __uint_as_float(r.w);
  }
};

// Part b of head h -> its rows in the sorted order, mb .. me (parts of REDUCE_ROWS rows, clusters in order).  By every lane of
// a wave.  False: the head has no such part.
__device__ __forceinline__ bool find_part(const ReduceCfg& cfg, int h, int b, int m, int lane, const int32_t* __restrict__ offs,
                                          int offs_stride, const int32_t* __restrict__ poff, const int32_t* __restrict__ pcl,
                                          int& mb, int& me) {
  const int32_t* po = poff + (size_t)h * offs_stride;
  const int32_t* of = offs + (size_t)h * offs_stride;
  int j, part, beg, end;
  if (m <= 128) {
    // few clusters: every lane takes two entries of both tables in one round trip and the
    // cluster of this part is found by a vote (j = number of clusters that start at or before b)
    const int a0 = lane, a1 = lane + 64;
    const int p0 = a0 <= m ? po[a0] : INT32_MAX, p1 = a1 <= m ? po[a1] : INT32_MAX;
    const int o0 = a0 <= m ? of[a0] : 0, o1 = a1 <= m ? of[a1] : 0;
    const int o2 = of[m], ptotal = po[m];
    if (b >= ptotal) return false;
    // entries 0..m-1 are cluster starts, entry m is the total
    const int cnt = __popcll(__ballot(a0 < m && p0 <= b)) + __popcll(__ballot(a1 < m && p1 <= b));
    j = cnt - 1;
    const int pj = j < 64 ? __shfl(p0, j) : __shfl(p1, j - 64);
    part = b - pj;
    beg = j < 64 ? __shfl(o0, j) : __shfl(o1, j - 64);
    const int jn = j + 1;
    end = jn == m ? o2 : (jn < 64 ? __shfl(o0, jn) : __shfl(o1, jn - 64));
  } else {
    if (b >= po[m]) return false;
    if (pcl) {
      j = pcl[(size_t)h * cfg.P + b];
    } else {
      int lo = 0, hi = m - 1;
      while (lo < hi) { const int mid = (lo + hi + 1) >> 1; if (po[mid] <= b) lo = mid; else hi = mid - 1; }
      j = lo;
    }
    part = b - po[j];
    beg = of[j]; end = of[j + 1];
  }
  mb = beg + part * REDUCE_ROWS;
  me = min(end, mb + REDUCE_ROWS);
  return true;
}

template <typename T, int D>
__global__ __launch_bounds__(64) void seg_reduce(const T* __restrict__ X, ReduceCfg cfg,
                                                 const int32_t* __restrict__ perm,
                                                 const int32_t* __restrict__ offs, int offs_stride,
                                                 const int32_t* __restrict__ poff, const int32_t* __restrict__ pcl,
                                                 float* __restrict__ psum, float* __restrict__ pnorm,
                                                 float* __restrict__ pmin, float* __restrict__ pmax) {
  constexpr int EV = Vec16<T>::N;     // elements per 16-byte load
  constexpr int LPR = D / EV;         // lanes per row
  constexpr int RPI = 64 / LPR;       // rows per wave step
  const int h = blockIdx.y, b = blockIdx.x;
  int m, mb, me;
  if (!reduce_setup(cfg, h, m)) return;
  const int lane = threadIdx.x, slot = lane / LPR, cl = lane % LPR;
  if (!find_part(cfg, h, b, m, lane, offs, offs_stride, poff, pcl, mb, me)) return;
  const int32_t* pm = perm + (size_t)h * cfg.N;
  const T* Xh = X + (size_t)h * cfg.N * D + cl * EV;
  float acc[EV], mn[EV], mx[EV];
#pragma unroll
  for (int e = 0; e < EV; ++e) { acc[e] = 0.f; mn[e] = INFINITY; mx[e] = -INFINITY; }
  float nsum = 0.f;
  auto add_row = [&](const float* x, bool valid) {
    float xs[EV];
#pragma unroll
    for (int e = 0; e < EV; ++e) xs[e] = x[e];
    if (cfg.normalize) {
      float ss = 0.f;
#pragma unroll
      for (int e = 0; e < EV; ++e) ss = fmaf(xs[e], xs[e], ss);
#pragma unroll
      for (int o = 1; o < LPR; o <<= 1) ss += __shfl_xor(ss, o);
      const float nrm = sqrtf(ss);
      const float inv = 1.0f / fmaxf(nrm, 1e-12f);
#pragma unroll
      for (int e = 0; e < EV; ++e) xs[e] *= inv;
      if (valid) nsum += nrm;
    }
    if (valid) {
#pragma unroll
      for (int e = 0; e < EV; ++e) {
        acc[e] += xs[e];
        if (cfg.want_box) { mn[e] = fminf(mn[e], xs[e]); mx[e] = fmaxf(mx[e], xs[e]); }
      }
    }
  };
  // The wave fetches up to 64 row indices with one coalesced load (the next 64 while the current
  // rows are summed), then keeps UNR row gathers in flight per lane: small clusters are bound by
  // the number of dependent memory round trips, not by bytes.  Every lane runs the same number of
  // steps (the shuffles in add_row need all lanes of a row present); rows past the end contribute
  // nothing.  The order in which a lane adds its rows is ascending, whatever UNR is.
  // The rows wait in registers as loaded (16 bytes, four registers each) and are decoded one by one when
  // they are added, so that sixteen gathers per lane fit where eight decoded rows did.
  constexpr int UNR = (64 / RPI) < 16 ? (64 / RPI) : 16;
  int idx_next = (mb + lane < me) ? pm[mb + lane] : 0;
  for (int r0 = mb; r0 < me; r0 += 64) {
    const int idx = idx_next;
    if (r0 + 64 < me) idx_next = (r0 + 64 + lane < me) ? pm[r0 + 64 + lane] : 0;
    const int nhere = min(64, me - r0);
    for (int k0 = 0; k0 < nhere; k0 += UNR * RPI) {
      uint4 raw[UNR];
      bool valid[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int k = k0 + u * RPI + slot;            // < 64 + RPI*UNR, but only k < nhere is used
        valid[u] = k < nhere;
        const int tok = __shfl(idx, k & 63);
        raw[u] = uint4{0u, 0u, 0u, 0u};
        if (valid[u]) raw[u] = *reinterpret_cast<const uint4*>(Xh + (size_t)tok * D);
      }
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        float x[EV];
        Vec16<T>::decode(raw[u], x);
        add_row(x, valid[u]);
      }
    }
  }
  // merge the row slots: slot s+o into slot s, o = RPI/2 ... 1
#pragma unroll
  for (int o = RPI / 2; o >= 1; o >>= 1) {
#pragma unroll
    for (int e = 0; e < EV; ++e) {
      acc[e] += __shfl_down(acc[e], o * LPR);
      mn[e] = fminf(mn[e], __shfl_down(mn[e], o * LPR));
      mx[e] = fmaxf(mx[e], __shfl_down(mx[e], o * LPR));
    }
    nsum += __shfl_down(nsum, o * LPR);
  }
  if (slot == 0) {
    const size_t o = (size_t)h * cfg.P + b;
#pragma unroll
    for (int e = 0; e < EV; ++e) {
      psum[o * D + cl * EV + e] = acc[e];
      if (cfg.want_box) { pmin[o * D + cl * EV + e] = mn[e]; pmax[o * D + cl * EV + e] = mx[e]; }
    }
    if (cfg.normalize && cl == 0) pnorm[o] = nsum;
  }
}

// The same sums, to the bit, for the fp32 query clustering in small launches: four waves a part, which load and normalise all
// of its rows at once and leave them in LDS; then a thread takes a column and the rows of one slot in ascending order, and
// the slots meet in the same tree.  A wave alone takes its part's rows in up to four dependent rounds and spends sixty
// instructions at half rate on every row it normalises: 318 parts, d=128, 26 us, here 14; 780 parts 31 and 18; d=64, 640
// parts 17 and 15.  From some 1 500 parts on the waves are enough (5 352: 55 us, here 131).
static constexpr int REDUCE_FEW = 1024;
template <int D>
__global__ __launch_bounds__(256) void seg_reduce_few(const float* __restrict__ X, ReduceCfg cfg,
                                                      const int32_t* __restrict__ perm,
                                                      const int32_t* __restrict__ offs, int offs_stride,
                                                      const int32_t* __restrict__ poff, const int32_t* __restrict__ pcl,
                                                      float* __restrict__ psum, float* __restrict__ pnorm) {
  constexpr int LPR = D / 4, RPI = 64 / LPR, STEPS = REDUCE_ROWS / (4 * RPI);
  static_assert(RPI * D == 256, "a thread a column and slot");
  const int h = blockIdx.y, b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int slot = lane / LPR, cl = lane % LPR;
  int m, mb, me;
  if (!reduce_setup(cfg, h, m)) return;
  if (!find_part(cfg, h, b, m, lane, offs, offs_stride, poff, pcl, mb, me)) return;
  __shared__ __attribute__((aligned(16))) float xs[REDUCE_ROWS][D];
  __shared__ float norms[REDUCE_ROWS];
  __shared__ float red[RPI][D];
  const int rows = me - mb;
  const int32_t* pm = perm + (size_t)h * cfg.N + mb;
  const float* Xh = X + (size_t)h * cfg.N * D + cl * 4;
  int tok[STEPS];
#pragma unroll
  for (int u = 0; u < STEPS; ++u) tok[u] = pm[min((u * 4 + wave) * RPI + slot, rows - 1)];
  float4 x[STEPS];
#pragma unroll
  for (int u = 0; u < STEPS; ++u) x[u] = *reinterpret_cast<const float4*>(Xh + (size_t)tok[u] * D);
#pragma unroll
  for (int u = 0; u < STEPS; ++u) {
    const int k = (u * 4 + wave) * RPI + slot;       // (rows past the end repeat the last one and are not summed)
    float ss = fmaf(x[u].x, x[u].x, 0.f);
    ss = fmaf(x[u].y, x[u].y, ss); ss = fmaf(x[u].z, x[u].z, ss); ss = fmaf(x[u].w, x[u].w, ss);
#pragma unroll
    for (int o = 1; o < LPR; o <<= 1) ss += __shfl_xor(ss, o);
    const float nrm = sqrtf(ss);
    const float inv = 1.0f / fmaxf(nrm, 1e-12f);
    if (cl == 0) norms[k] = nrm;
    *reinterpret_cast<float4*>(&xs[k][cl * 4]) = float4{x[u].x * inv, x[u].y * inv, x[u].z * inv, x[u].w * inv};
  }
  __syncthreads();
  {
    const int col = tid % D, s = tid / D;
    float acc = 0.f;
#pragma unroll 8
    for (int r = s; r < rows; r += RPI) acc += xs[r][col];
    red[s][col] = acc;
  }
  if (tid < RPI) {                                   // norms: a slot a lane, then the slots
    float ns = 0.f;
#pragma unroll 8
    for (int r = tid; r < rows; r += RPI) ns += norms[r];
#pragma unroll
    for (int o = RPI / 2; o >= 1; o >>= 1) ns += __shfl_down(ns, o);
    if (tid == 0) pnorm[(size_t)h * cfg.P + b] = ns;
  }
  __syncthreads();
  if (tid >= D) return;
  float a[RPI];
#pragma unroll
  for (int s = 0; s < RPI; ++s) a[s] = red[s][tid];
#pragma unroll
  for (int o = RPI / 2; o >= 1; o >>= 1)
#pragma unroll
    for (int s = 0; s < o; ++s) a[s] += a[s + o];
  psum[((size_t)h * cfg.P + b) * D + tid] = a[0];
}

// Combine the parts and write centres.
//   update_assign = 1 (Lloyd step): non-empty clusters get master := mean (or unit mean), where it is kept, the
//     I/O-dtype copy used by the next assignment, its fp32 image and the arg-max bias.
//   update_assign = 0 (final): out_cent := mean / unit mean (empty: `fallback` row), sizes, mean
//     norms, boxes.  `master` is also refreshed when given (query clustering returns it).
struct FinalizeCfg {
  int mode; int m_const; int P; int m_bound; int cap; int master_stride;
  const KState* st;
  int spherical; int update_assign; int lp_is_bf16; int want_box;
  const int32_t* bcnt; int nb_stride;     // block sums of the assignment kernel instead of cluster parts (stage mode)
  int blk_points;                         // points of a block; 0: nb_stride blocks (walks of the one-read query pass), whatever the state says
  StateExport ex;                         // the last launch of a key clustering: what it leaves of its state (home NULL: nothing)
};

// The state of a head as later steps and calls find it in `home` (mode 1, a warm start: its one pseudo-stage is over), and
// the outputs that are copies of it.  By the first wave of a head's first workgroup; `home` is not the array that the
// others read, or is left as it is.
__device__ __forceinline__ void export_state(const StateExport& ex, const KState* __restrict__ st, int mode, int h, int lane) {
  constexpr int W = sizeof(KState) / 4, OFFS = offsetof(KState, stage_offs) / 4;
  static_assert(W <= 64, "a word a lane");
  const KState& s = st[h];
  const int m = s.m_t;
  int v = lane < W ? reinterpret_cast<const int32_t*>(&s)[lane] : 0;
  if (mode == 1) {
    if (lane == offsetof(KState, ucount) / 4 || lane == offsetof(KState, active) / 4) v = 0;
    if (lane == offsetof(KState, stage) / 4 || lane == offsetof(KState, done) / 4) v = 1;
    if (lane == offsetof(KState, ccount) / 4 || lane == OFFS + 1) v = m;
  }
  if (ex.home != st && lane < W) reinterpret_cast<int32_t*>(&ex.home[h])[lane] = v;
  const int ccount = mode == 1 ? m : s.ccount, stage = mode == 1 ? 1 : s.stage;
  if (lane == 0) {
    if (h == 0 && ex.tau_used) ex.tau_used[0] = ex.tau[0];
    if (ex.k_count) ex.k_count[h] = ccount;
    if (ex.full_flag) ex.full_flag[h] = s.full;
  }
  const int i = lane - OFFS;
  if (ex.stage_offs && i >= 0 && i <= ADACLUSTER_MAX_STAGES)
    ex.stage_offs[(size_t)h * (ADACLUSTER_MAX_STAGES + 1) + i] = i <= stage ? v : ccount;
}

constexpr int FIN_ROWS = 4;           // clusters per workgroup, one wave each (no step needs the workgroup)
template <int D>
__global__ __launch_bounds__(64 * FIN_ROWS) void finalize_centroids(FinalizeCfg cfg, const int32_t* __restrict__ offs,
                                                         int offs_stride, const int32_t* __restrict__ poff,
                                                         const float* __restrict__ psum,
                                                         const float* __restrict__ pnorm,
                                                         const float* __restrict__ pmin,
                                                         const float* __restrict__ pmax,
                                                         float* __restrict__ master, void* __restrict__ assign_lp,
                                                         float* __restrict__ assign_f32, float* __restrict__ bias,
                                                         float* __restrict__ out_cent, const float* __restrict__ fallback,
                                                         int32_t* __restrict__ out_sizes, float* __restrict__ out_mean_norm,
                                                         float* __restrict__ out_bmin, float* __restrict__ out_bmax) {
  constexpr int CPL = D / 64;          // columns per lane
  const int h = blockIdx.y, j = blockIdx.x * FIN_ROWS + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (cfg.ex.home && blockIdx.x == 0 && threadIdx.x < 64) export_state(cfg.ex, cfg.st, cfg.mode, h, lane);
  int m, row_off = 0;
  if (cfg.mode == 0) m = cfg.m_const;
  else {
    const KState& s = cfg.st[h];
    if (cfg.mode == 1) { if (!s.active) return; m = s.m_t; row_off = s.ccount; }
    else m = s.ccount;
  }
  if (j >= m) {
    if (!cfg.update_assign && out_sizes && j < cfg.cap) out_sizes[(size_t)h * cfg.cap + j] = 0;
    return;
  }
  int nj, p_beg, p_end;
  if (cfg.bcnt) {
    // the workgroups of stage_pass, or the walks of qpass_mfma, in order
    const int nb = cfg.blk_points > 0 ? (cfg.st[h].ucount + cfg.blk_points - 1) / cfg.blk_points : cfg.nb_stride;
    nj = 0;
    for (int b = lane; b < nb; b += 64) nj += cfg.bcnt[((size_t)h * cfg.nb_stride + b) * ACC_MAXM + j];
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) nj += __shfl_xor(nj, o);
    p_beg = j * cfg.nb_stride; p_end = p_beg + nb;
  } else {
    nj = offs[(size_t)h * offs_stride + j + 1] - offs[(size_t)h * offs_stride + j];
    p_beg = poff[(size_t)h * offs_stride + j]; p_end = poff[(size_t)h * offs_stride + j + 1];
  }
  const size_t pbase = (size_t)h * cfg.P;
  float s[CPL], mn[CPL], mx[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) { s[q] = 0.f; mn[q] = INFINITY; mx[q] = -INFINITY; }
  float ns = 0.f;
  int p = p_beg;
  if (!cfg.want_box && (!cfg.spherical || cfg.update_assign)) {
    // sums only: eight parts' loads in flight, added in part order all the same
    for (; p + 8 <= p_end; p += 8) {
      float t[8][CPL];
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int q = 0; q < CPL; ++q) t[u][q] = psum[(pbase + p + u) * D + lane + 64 * q];
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int q = 0; q < CPL; ++q) s[q] += t[u][q];
    }
  }
  for (; p < p_end; ++p) {
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      s[q] += psum[(pbase + p) * D + lane + 64 * q];
      if (cfg.want_box) {
        mn[q] = fminf(mn[q], pmin[(pbase + p) * D + lane + 64 * q]);
        mx[q] = fmaxf(mx[q], pmax[(pbase + p) * D + lane + 64 * q]);
      }
    }
    if (cfg.spherical && !cfg.update_assign) ns += pnorm[pbase + p];     // (member norms matter to the final outputs only)
  }
  bool ok = nj > 0;
  float val[CPL];
  if (cfg.spherical) {
    float ss = 0.f;
#pragma unroll
    for (int q = 0; q < CPL; ++q) ss = fmaf(s[q], s[q], ss);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) ss += __shfl_xor(ss, o);
    const float nrm = sqrtf(ss);
    ok = ok && (nrm >= 1e-12f);
#pragma unroll
    for (int q = 0; q < CPL; ++q) val[q] = s[q] / fmaxf(nrm, 1e-30f);
  } else {
#pragma unroll
    for (int q = 0; q < CPL; ++q) val[q] = s[q] / (float)max(nj, 1);
  }
  if (cfg.update_assign) {
    if (!ok) return;
    float bsum = 0.f;
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      const int col = lane + 64 * q;
      if (master) master[((size_t)h * cfg.master_stride + j) * D + col] = val[q];
      const size_t ao = ((size_t)h * cfg.cap + row_off + j) * D + col;
      float img = val[q];
      if (cfg.lp_is_bf16) {
        const bf16raw r = f32_to_bf16(val[q]);
        reinterpret_cast<bf16raw*>(assign_lp)[ao] = r;
        img = bf16_to_f32(r);
      } else {
        reinterpret_cast<float*>(assign_lp)[ao] = img;
      }
      assign_f32[ao] = img;
      bsum = fmaf(img, img, bsum);
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) bsum += __shfl_xor(bsum, o);
    if (lane == 0) bias[(size_t)h * cfg.cap + row_off + j] = cfg.spherical ? 0.f : -0.5f * bsum;
    return;
  }
  // final outputs
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    const int col = lane + 64 * q;
    const size_t oo = ((size_t)h * cfg.cap + j) * D + col;
    if (ok) {
      out_cent[oo] = val[q];
    } else if (fallback) {
      out_cent[oo] = fallback[oo];
    }
    if (cfg.want_box) {
      out_bmin[oo] = nj > 0 ? mn[q] : 0.f;
      out_bmax[oo] = nj > 0 ? mx[q] : 0.f;
    }
  }
  if (lane == 0) {
    if (out_sizes) out_sizes[(size_t)h * cfg.cap + j] = nj;
    // mean member norm, the factor that brings unit-centroid scores back to logits; 1 for raw centroids
    if (out_mean_norm) out_mean_norm[(size_t)h * cfg.cap + j] = nj > 0 ? (cfg.spherical ? ns / (float)nj : 1.f) : 0.f;
  }
}

// ------------------------------------------------------------------------------------------
// Label sort and final member statistics of short heads in one launch
// ------------------------------------------------------------------------------------------
// A workgroup is a cluster: it reads all labels of the head, so it knows how many items come before its own and which those
// are, in order.  That is its part of the sorted order and of the offsets; it sums its rows, in parts of REDUCE_ROWS, a wave
// each, and writes what finalize_centroids writes with update_assign = 0: the order of all sums is that of seg_reduce and
// finalize_centroids, and so are the results, to the bit.
// Bound by latency: three dependent trips to memory and the sums, 8-9 us, in the place of a sort by one workgroup (10-14 us), a
// reduction (7-10) and a combining launch (3-4).  cluster_stats_fits() has the line.
struct StatsCfg {
  int mode; int m_const; int N; int cap;        // mode as FinalizeCfg
  const KState* st;
  int spherical; int want_box;
  StateExport ex;
};
constexpr int STATS_NT = 512, STATS_ITEMS = 4096;
template <typename T, int D>
__global__ __launch_bounds__(STATS_NT) void cluster_stats(const T* __restrict__ X, StatsCfg cfg, const int32_t* __restrict__ labels,
                                                          int32_t* __restrict__ perm, int32_t* __restrict__ offs, int offs_stride,
                                                          float* __restrict__ out_cent, const float* __restrict__ fallback,
                                                          int32_t* __restrict__ out_sizes, float* __restrict__ out_mean_norm,
                                                          float* __restrict__ out_bmin, float* __restrict__ out_bmax) {
  constexpr int EV = Vec16<T>::N, LPR = D / EV, RPI = 64 / LPR, NW = STATS_NT / 64, PER = STATS_ITEMS / STATS_NT, CPL = D / 64;
  constexpr int UNR = (REDUCE_ROWS / RPI) < 16 ? REDUCE_ROWS / RPI : 16, MAXP = STATS_ITEMS / REDUCE_ROWS;
  const int h = blockIdx.y, j = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // this thread's labels: positions wave * 64 * PER + 64 i + lane
  const int n = cfg.N;
  const int32_t* lab = labels + (size_t)h * n;
  int l[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) { const int pos = (wave * PER + i) * 64 + lane; l[i] = pos < n ? lab[pos] : -1; }
  if (cfg.ex.home && j == 0 && wave == 0) export_state(cfg.ex, cfg.st, cfg.mode, h, lane);
  const int m = cfg.mode == 0 ? cfg.m_const : cfg.mode == 1 ? cfg.st[h].m_t : cfg.st[h].ccount;
  int32_t* const of = offs + (size_t)h * offs_stride;
  if (j == 0) {
    if (out_sizes) for (int i = m + tid; i < cfg.cap; i += STATS_NT) out_sizes[(size_t)h * cfg.cap + i] = 0;
    if (m == 0 && tid == 0) of[0] = 0;
  }
  if (j >= m) return;
  __shared__ int32_t list[STATS_ITEMS];
  __shared__ int32_t whit[NW], wless[NW];
  __shared__ float psum[MAXP][D], pnorm[MAXP], wmin[NW][D], wmax[NW][D];
  const uint64_t below = (1ull << lane) - 1ull;
  int mine = 0, less = 0, at[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const uint64_t b = __ballot(l[i] == j);
    at[i] = mine + __popcll(b & below);
    mine += __popcll(b);
    less += __popcll(__ballot((uint32_t)l[i] < (uint32_t)j));
  }
  if (lane == 0) { whit[wave] = mine; wless[wave] = less; }
  __syncthreads();
  int base = 0, nj = 0, start = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) { const int c = whit[w]; if (w < wave) base += c; nj += c; start += wless[w]; }
#pragma unroll
  for (int i = 0; i < PER; ++i) if (l[i] == j) list[base + at[i]] = (wave * PER + i) * 64 + lane;
  __syncthreads();
  for (int i = tid; i < nj; i += STATS_NT) perm[(size_t)h * n + start + i] = list[i];
  if (tid == 0) { of[j] = start; if (j == m - 1) of[m] = start + nj; }
  const int slot = lane / LPR, cl = lane % LPR, parts = (nj + REDUCE_ROWS - 1) / REDUCE_ROWS;
  const T* Xh = X + (size_t)h * n * D + cl * EV;
  float mn[EV], mx[EV];
#pragma unroll
  for (int e = 0; e < EV; ++e) { mn[e] = INFINITY; mx[e] = -INFINITY; }
  for (int p = wave; p < parts; p += NW) {
    const int me = min(nj, (p + 1) * REDUCE_ROWS);
    float acc[EV], nsum = 0.f;
#pragma unroll
    for (int e = 0; e < EV; ++e) acc[e] = 0.f;
    for (int i0 = p * REDUCE_ROWS; i0 < me; i0 += UNR * RPI) {
      uint4 raw[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int i = i0 + u * RPI + slot;
        raw[u] = uint4{0u, 0u, 0u, 0u};
        if (i < me) raw[u] = *reinterpret_cast<const uint4*>(Xh + (size_t)list[i] * D);
      }
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const bool valid = i0 + u * RPI + slot < me;
        float x[EV];
        Vec16<T>::decode(raw[u], x);
        if (cfg.spherical) {
          float ss = 0.f;
#pragma unroll
          for (int e = 0; e < EV; ++e) ss = fmaf(x[e], x[e], ss);
#pragma unroll
          for (int o = 1; o < LPR; o <<= 1) ss += __shfl_xor(ss, o);
          const float nrm = sqrtf(ss), inv = 1.0f / fmaxf(nrm, 1e-12f);
#pragma unroll
          for (int e = 0; e < EV; ++e) x[e] *= inv;
          if (valid) nsum += nrm;
        }
        if (valid) {
#pragma unroll
          for (int e = 0; e < EV; ++e) {
            acc[e] += x[e];
            if (cfg.want_box) { mn[e] = fminf(mn[e], x[e]); mx[e] = fmaxf(mx[e], x[e]); }
          }
        }
      }
    }
#pragma unroll
    for (int o = RPI / 2; o >= 1; o >>= 1) {
#pragma unroll
      for (int e = 0; e < EV; ++e) acc[e] += __shfl_down(acc[e], o * LPR);
      nsum += __shfl_down(nsum, o * LPR);
    }
    if (slot == 0) {
#pragma unroll
      for (int e = 0; e < EV; ++e) psum[p][cl * EV + e] = acc[e];
      if (cl == 0) pnorm[p] = nsum;
    }
  }
  if (cfg.want_box) {
#pragma unroll
    for (int o = RPI / 2; o >= 1; o >>= 1)
#pragma unroll
      for (int e = 0; e < EV; ++e) {
        mn[e] = fminf(mn[e], __shfl_down(mn[e], o * LPR));
        mx[e] = fmaxf(mx[e], __shfl_down(mx[e], o * LPR));
      }
    if (slot == 0) {
#pragma unroll
      for (int e = 0; e < EV; ++e) { wmin[wave][cl * EV + e] = mn[e]; wmax[wave][cl * EV + e] = mx[e]; }
    }
  }
  __syncthreads();
  if (wave > 0) return;
  float s[CPL], ss = 0.f, ns = 0.f;
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    s[q] = 0.f;
    for (int p = 0; p < parts; ++p) s[q] += psum[p][lane + 64 * q];
    ss = fmaf(s[q], s[q], ss);
  }
  bool ok = nj > 0;
  float div = (float)max(nj, 1);
  if (cfg.spherical) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) ss += __shfl_xor(ss, o);
    const float nrm = sqrtf(ss);
    ok = ok && nrm >= 1e-12f;
    div = fmaxf(nrm, 1e-30f);
    for (int p = 0; p < parts; ++p) ns += pnorm[p];
  }
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    const int cq = lane + 64 * q;
    const size_t oo = ((size_t)h * cfg.cap + j) * D + cq;
    if (ok) out_cent[oo] = s[q] / div;
    else if (fallback) out_cent[oo] = fallback[oo];
    if (cfg.want_box) {
      float lo = wmin[0][cq], hi = wmax[0][cq];
#pragma unroll
      for (int w = 1; w < NW; ++w) { lo = fminf(lo, wmin[w][cq]); hi = fmaxf(hi, wmax[w][cq]); }
      out_bmin[oo] = nj > 0 ? lo : 0.f;
      out_bmax[oo] = nj > 0 ? hi : 0.f;
    }
  }
  if (lane == 0) {
    if (out_sizes) out_sizes[(size_t)h * cfg.cap + j] = nj;
    if (out_mean_norm) out_mean_norm[(size_t)h * cfg.cap + j] = nj > 0 ? (cfg.spherical ? ns / (float)nj : 1.f) : 0.f;
  }
}

// ------------------------------------------------------------------------------------------
// Centroid update of a stage with few points in ONE launch (fp32 inputs): the workgroup of a centre finds
// its members in the label list itself (an ordered compaction, so the member order is the list order),
// sums their rows in a fixed order and writes the new centre, its copies for the assignment kernel and
// the arg-max bias.  It stands for the label sort, the segmented reduction and the combining kernel,
// three launches that are each bound by latency at a few thousand points.
// ------------------------------------------------------------------------------------------
constexpr int DIRECT_ROUND = 4096;          // list positions scanned per round: 1024 per wave, 16 per lane
constexpr long long DIRECT_MAX_VISITS = 1 << 21;
constexpr int DIRECT_MAX_POINTS = 4 * DIRECT_ROUND;  // a workgroup scans the list alone: at most four rounds   // centres x points up to which every centre scans the whole list

template <int D>
__global__ __launch_bounds__(256) void update_direct_f32(const float* __restrict__ X, int N, int cap, int master_stride,
                                                         const KState* __restrict__ st,
                                                         const int32_t* __restrict__ labels,
                                                         const int32_t* __restrict__ ulist,
                                                         float* __restrict__ master, float* __restrict__ assign_lp,
                                                         float* __restrict__ assign_f32, float* __restrict__ bias) {
  constexpr int LPR = D / 4, G = 256 / LPR;   // lanes per row (16 bytes each), rows in flight per step
  const int h = blockIdx.y, j = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const KState& s = st[h];
  if (!s.active) return;
  const int n = s.ucount, m = s.m_t, row_off = s.ccount;
  if (j >= m) return;
  __shared__ int32_t list[DIRECT_ROUND];
  __shared__ int32_t wcnt[4];
  __shared__ float4 red[256];
  const int32_t* lab = labels + (size_t)h * N;
  const int32_t* ul = ulist ? ulist + (size_t)h * N : nullptr;
  const float* Xh = X + (size_t)h * N * D;
  const int g = tid / LPR, cl = tid % LPR;
  const uint64_t below = (1ull << lane) - 1ull;
  float4 acc = {0.f, 0.f, 0.f, 0.f};
  int total = 0;
  for (int r0 = 0; r0 < n; r0 += DIRECT_ROUND) {
    // wave w scans positions r0 + 1024 w ... in 16 steps of 64; members keep their list order
    int tok[16];
    uint32_t hit = 0;
    int mine = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int pos = r0 + wave * 1024 + i * 64 + lane;
      const bool in = pos < n;
      const int l = in ? lab[pos] : -1;
      tok[i] = in ? (ul ? ul[pos] : pos) : 0;
      if (l == j) hit |= 1u << i;
    }
    int woff[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const uint64_t b = __ballot((hit >> i) & 1u);
      woff[i] = mine + __popcll(b & below);
      mine += __popcll(b);
    }
    __syncthreads();                 // the list of the round before has been summed
    if (lane == 0) wcnt[wave] = mine;
    __syncthreads();
    int base = 0, cnt = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) { const int c = wcnt[w]; if (w < wave) base += c; cnt += c; }
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if ((hit >> i) & 1u) list[base + woff[i]] = tok[i];
    __syncthreads();
    // row i of the round goes to row group i % G; a group adds its rows in ascending order
    for (int i0 = g; i0 < cnt; i0 += 4 * G) {
      float4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + u * G;
        v[u] = float4{0.f, 0.f, 0.f, 0.f};
        if (i < cnt) v[u] = *reinterpret_cast<const float4*>(Xh + (size_t)list[i] * D + cl * 4);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) { acc.x += v[u].x; acc.y += v[u].y; acc.z += v[u].z; acc.w += v[u].w; }
    }
    total += cnt;
  }
  if (total == 0) return;            // an empty cluster keeps its centre
  red[tid] = acc;
  __syncthreads();
  if (tid >= LPR) return;
  float4 sum = red[cl];
#pragma unroll
  for (int q = 1; q < G; ++q) {
    const float4 t = red[q * LPR + cl];
    sum.x += t.x; sum.y += t.y; sum.z += t.z; sum.w += t.w;
  }
  const float cntf = (float)total;
  const float4 val = {sum.x / cntf, sum.y / cntf, sum.z / cntf, sum.w / cntf};
  if (master) *reinterpret_cast<float4*>(master + ((size_t)h * master_stride + j) * D + cl * 4) = val;
  const size_t ao = ((size_t)h * cap + row_off + j) * D + cl * 4;
  *reinterpret_cast<float4*>(assign_lp + ao) = val;
  *reinterpret_cast<float4*>(assign_f32 + ao) = val;
  float bsum = fmaf(val.x, val.x, 0.f);
  bsum = fmaf(val.y, val.y, bsum); bsum = fmaf(val.z, val.z, bsum); bsum = fmaf(val.w, val.w, bsum);
#pragma unroll
  for (int o = 1; o < LPR; o <<= 1) bsum += __shfl_xor(bsum, o);
  if (cl == 0) bias[(size_t)h * cap + row_off + j] = -0.5f * bsum;
}

// Initial centres: of the query clustering a strided sample of all points or (warm start) the rows that `master` holds, and
// of a warm-started key clustering (Sec. 3.2.2, "Efficient initialization": one pseudo-stage over all tokens, the centre
// count given) the rows of `master`; that launch (`warm`) also opens the state of every head.  A wave a centre.  (A stage of
// Algorithm 1 takes its sample in stage_open.)
struct WarmStart { KState* st; const int32_t* k_count; const int32_t* full_flag; };
constexpr int INIT_ROWS = 4;
template <typename T, int D>
__global__ __launch_bounds__(64 * INIT_ROWS) void init_centroids(const T* __restrict__ X, int N, int m_const, WarmStart warm,
                                                     int spherical, int source_master, int cap, int master_stride,
                                                     int lp_is_bf16, float* __restrict__ master,
                                                     void* __restrict__ assign_lp, float* __restrict__ assign_f32,
                                                     float* __restrict__ bias) {
  constexpr int CPL = D / 64;
  const int h = blockIdx.y, j = blockIdx.x * INIT_ROWS + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  int m = m_const;
  if (warm.st) {
    m = max(1, min(min(warm.k_count[h], cap), N));
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      KState s{};
      s.ucount = N; s.m_t = m; s.full = warm.full_flag[h] != 0; s.active = 1; s.u_hist[0] = N;
      warm.st[h] = s;
    }
  }
  if (j >= m) return;
  float val[CPL];
  if (source_master) {
#pragma unroll
    for (int q = 0; q < CPL; ++q) val[q] = master[((size_t)h * master_stride + j) * D + lane + 64 * q];
  } else {
    const int tok = sample_at(j, N, m);
    const T* row = X + ((size_t)h * N + tok) * D;
#pragma unroll
    for (int q = 0; q < CPL; ++q) val[q] = Elem<T>::load(row + lane + 64 * q);
    if (spherical) {
      float ss = 0.f;
#pragma unroll
      for (int q = 0; q < CPL; ++q) ss = fmaf(val[q], val[q], ss);
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) ss += __shfl_xor(ss, o);
      const float inv = 1.0f / fmaxf(sqrtf(ss), 1e-12f);
#pragma unroll
      for (int q = 0; q < CPL; ++q) val[q] *= inv;
    }
  }
  float bsum = 0.f;
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    const int col = lane + 64 * q;
    master[((size_t)h * master_stride + j) * D + col] = val[q];
    const size_t ao = ((size_t)h * cap + j) * D + col;
    float img = val[q];
    if (lp_is_bf16) {
      const bf16raw r = f32_to_bf16(val[q]);
      reinterpret_cast<bf16raw*>(assign_lp)[ao] = r;
      img = bf16_to_f32(r);
    } else {
      reinterpret_cast<float*>(assign_lp)[ao] = img;
    }
    assign_f32[ao] = img;
    bsum = fmaf(img, img, bsum);
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) bsum += __shfl_xor(bsum, o);
  if (lane == 0) bias[(size_t)h * cap + j] = spherical ? 0.f : -0.5f * bsum;
}

// ------------------------------------------------------------------------------------------
// Algorithm 1 bookkeeping
// ------------------------------------------------------------------------------------------
// tau = factor x mean first-stage distance over all heads and tokens (Sec. 4.1), from the sums that the last pass of the
// first stage left per workgroup.  Called by a whole workgroup; a fixed order: thread i takes elements i, i + NT, ..., then
// a fixed tree.
struct TauCfg { const double* part; int count; double denom; float factor; float* out /* [0] = tau, [1] = tau^2 */; };
template <int NT>
__device__ __forceinline__ float tau_of(const TauCfg& c) {
  const int tid = threadIdx.x;
  double s = 0.0;
  for (int i = tid; i < c.count; i += 4 * NT) {
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = i + u * NT < c.count ? c.part[i + u * NT] : 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u) s += v[u];
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) s += __shfl_xor(s, o);
  __shared__ double ws[NT / 64];
  if ((tid & 63) == 0) ws[tid >> 6] = s;
  __syncthreads();
  double tot = 0.0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) tot += ws[w];
  return (float)((double)c.factor * tot / c.denom);
}
__global__ __launch_bounds__(1024) void tau_final(TauCfg c) {
  const float tau = tau_of<1024>(c);
  if (threadIdx.x == 0) { c.out[0] = tau; c.out[1] = tau * tau; }
}

__global__ void tau_set(float tau, float* __restrict__ tau_out) {
  if (threadIdx.x == 0 && blockIdx.x == 0) { tau_out[0] = tau; tau_out[1] = tau * tau; }
}

// Threshold filter of Algorithm 1: tokens with d < tau leave U.  Survivors per KEEP_ITEMS points of the first stage, whose
// threshold is known only after its last pass (a later stage's last pass counts them itself).
constexpr int KEEP_ITEMS = 1024;
// Up to TAU_SUMS sums every workgroup forms the threshold itself, in the same order (tc.part; NULL: tau holds it): the
// launch between the two cost 4-5 us and this costs one trip to the L2.
constexpr int TAU_SUMS = 4096;
__global__ __launch_bounds__(256) void keep_count(const KState* __restrict__ st, const float* __restrict__ dist2, int N,
                                                  TauCfg tc, const float* __restrict__ tau, int32_t* __restrict__ cnt, int cnt_stride,
                                                  int32_t* __restrict__ surv, int32_t* __restrict__ stage_of) {
  const int h = blockIdx.y, b = blockIdx.x, tid = threadIdx.x;
  float t2;
  if (tc.part) {
    const float t = tau_of<256>(tc);
    t2 = t * t;
    if (h == 0 && b == 0 && tid == 0) { tc.out[0] = t; tc.out[1] = t2; }
  } else t2 = tau[1];
  const KState& s = st[h];
  if (!s.active) return;
  const int n = s.ucount;
  constexpr int IPT = KEEP_ITEMS / 256;
  const int p0 = b * KEEP_ITEMS + tid * IPT, lane = tid & 63, wave = tid >> 6;
  bool keep[IPT];
  int c = 0;
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int p = p0 + i;
    keep[i] = p < n && !(dist2[(size_t)h * N + p] < t2);
    c += keep[i] ? 1 : 0;
  }
  int incl = c;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) { const int v = __shfl_up(incl, o); if (lane >= o) incl += v; }
  __shared__ int32_t ws[4];
  if (lane == 63) ws[wave] = incl;
  __syncthreads();
  if (tid == 0) cnt[(size_t)h * cnt_stride + b] = ws[0] + ws[1] + ws[2] + ws[3];
  if (!surv) return;
  // the survivors too, for the pass that opens the next stage (the first stage's positions are tokens)
  int at = b * KEEP_ITEMS + incl - c;
#pragma unroll
  for (int w = 0; w < 4; ++w) if (w < wave) at += ws[w];
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    if (keep[i]) surv[(size_t)h * N + at++] = p0 + i;
    else if (stage_of && p0 + i < n) stage_of[(size_t)h * N + p0 + i] = 0;
  }
}

// Between two stages of Algorithm 1, in one launch: the threshold filter of the stage that ends, the head of the
// while-loop (U empty?  |C| >= N_max, flag F?  stage and leftover limits; then the centre count m_t), and the initial
// centres of the stage that opens, a strided sample of the U being written.  Nothing waits for another workgroup: the
// survivors were counted per `items` points, so every workgroup sums those counts for itself and knows the new |U|,
// the loop's decision, where its own points go (the first `nblk` workgroups) or which point is the j-th survivor (the
// next, a wave per centre).  The state is read from `in` and written, by the last workgroup of a head, which has no points and
// no centres, to `out`, another array.  The last head to report writes {active heads, max |U|, max m_t, epoch} to `report`.
// Stages of block sums are opened by their first pass instead (stage_pass).  Bound by launch latency and five dependent trips to
// the L2: 8-10 us.  In three launches (the filter by one workgroup per
// head 13-27 us, the loop head 4, the centres 4) and with an event for the host behind the second, a late stage of
// 30 x 5 000 points took 68 us in all; it takes 47.
template <typename T, int D>
__global__ __launch_bounds__(256) void stage_open(const T* __restrict__ X, OpenCfg c) {
  constexpr int CPL = D / 64;
  const int h = blockIdx.y, bx = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  NewState s;
  __shared__ int32_t wtot[4], s_before, s_blk[4], s_rank[4];
  int total = c.N, ex = 0, mine = 0, b0 = 0, b1 = 0, n = c.N;
  const int32_t* cnt = c.cnt + (size_t)h * c.cnt_stride;
  // this thread's points, where the workgroup moves survivors
  constexpr int IPT = KEEP_ITEMS / 256;
  const float* dh = c.dist2 + (size_t)h * c.N;
  const int ipt = c.items >> 8 ? c.items >> 8 : 1, p0 = bx * c.items + tid * ipt;
  const bool has = tid * ipt < c.items;
  float d2[IPT]; int tok_in[IPT];
  if (c.first) {
    s.ucount = c.N; s.ccount = 0; s.m_t = 0; s.stage = 0; s.done = 0; s.full = 0;
    if (c.sums && h == 0 && bx == 0 && tid < 4) c.sums[tid] = 0;
  } else {
    const KState& o = c.in[h];
    const int c0 = cnt[min(tid, c.cnt_stride - 1)];          // (ahead of the state: one trip for both)
    if (!o.active) {               // closed before: carried over
      if (bx == (int)gridDim.x - 1) carry_state(c, h, tid);
      return;
    }
    s.ucount = o.ucount; s.ccount = o.ccount; s.m_t = o.m_t; s.stage = o.stage; s.full = o.full; s.done = 0;
    n = min(s.ucount, c.N);
    const int nb = (n + c.items - 1) / c.items;
    if (bx < c.nblk) {
      if (bx >= nb) return;
#pragma unroll
      for (int i = 0; i < IPT; ++i) {
        const int p = p0 + i;
        const bool valid = has && i < ipt && p < n;
        d2[i] = dh[valid ? p : 0];
        tok_in[i] = valid ? (c.uin ? c.uin[(size_t)h * c.N + p] : p) : -1;
      }
    }
    int before = 0;
    if (nb <= 256) {
      b0 = min(nb, tid); b1 = min(nb, tid + 1);
      mine = tid < nb ? c0 : 0;
    } else {
      const int per = (nb + 255) / 256;
      b0 = min(nb, tid * per); b1 = min(nb, b0 + per);
      for (int b = b0; b < b1; ++b) { const int v = cnt[b]; mine += v; before += b < bx ? v : 0; }
    }
    int incl = mine;
#pragma unroll
    for (int o2 = 1; o2 < 64; o2 <<= 1) { const int v = __shfl_up(incl, o2); if (lane >= o2) incl += v; }
    if (lane == 63) wtot[wave] = incl;
    __syncthreads();
    total = 0;
    ex = incl - mine;
#pragma unroll
    for (int w = 0; w < 4; ++w) { const int v = wtot[w]; if (w < wave) ex += v; total += v; }
    if (bx >= b0 && bx < b1) s_before = ex + before;
    s.ucount = total; s.ccount += s.m_t; s.stage += 1;
  }
  loop_head(s, c.N, c.n_max, c.m0, c.m_min, c.max_stages, c.u_min);
  if (bx == (int)gridDim.x - 1) { write_state(c, h, tid, s); return; }      // (one more than moves points or forms centres)

  if (bx < c.nblk) {               // the survivors of this workgroup's points move up, in order
    __syncthreads();
    const float t2 = c.tau[1];
    bool keep[IPT]; int k = 0;
#pragma unroll
    for (int i = 0; i < IPT; ++i) { keep[i] = tok_in[i] >= 0 && !(d2[i] < t2); k += keep[i] ? 1 : 0; }
    int incl = k;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) { const int v = __shfl_up(incl, o); if (lane >= o) incl += v; }
    const int before = s_before;
    __syncthreads();               // every thread has its use of the wave totals behind it
    if (lane == 63) wtot[wave] = incl;
    __syncthreads();
    int pos = before + incl - k;
#pragma unroll
    for (int w = 0; w < 4; ++w) if (w < wave) pos += wtot[w];
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
      if (keep[i]) c.uout[(size_t)h * c.N + pos++] = tok_in[i];
      else if (tok_in[i] >= 0 && c.stage_of) c.stage_of[(size_t)h * c.N + tok_in[i]] = c.stage;
    }
    return;
  }

  // initial centre j: survivor number floor((2j+1)|U| / 2m)
  const int j0 = (bx - c.nblk) * 4, j = j0 + wave;
  if (!s.active || j0 >= s.m_t) return;
  int tok = sample_at(j, total, s.m_t);
  if (!c.first) {
#pragma unroll
    for (int w = 0; w < 4; ++w) {  // the thread whose run of counts holds it says in which count and how far into it
      const int q = sample_at(j0 + w, total, s.m_t);
      if (j0 + w < s.m_t && q >= ex && q < ex + mine) {
        int b = b0, left = q - ex;
        for (; left >= cnt[b]; ++b) left -= cnt[b];
        s_blk[w] = b; s_rank[w] = left;
      }
    }
    __syncthreads();
    if (j >= s.m_t) return;
    const float t2 = c.tau[1];
    const int base = s_blk[wave] * c.items;
    int left = s_rank[wave], at = -1;
    for (int q0 = 0; q0 < c.items && at < 0; q0 += 256) {      // 256 points at a time, their loads together
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = dh[min(base + q0 + 64 * u + lane, n - 1)];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int p = base + q0 + 64 * u + lane;
        const uint64_t mask = __ballot(q0 + 64 * u < c.items && p < n && !(v[u] < t2));
        const int here = __popcll(mask);
        if (at < 0 && left < here) {
          const bool it = ((mask >> lane) & 1) && __popcll(mask & (lane ? ~0ull >> (64 - lane) : 0ull)) == left;
          at = base + q0 + 64 * u + __ffsll((unsigned long long)__ballot(it)) - 1;
        }
        left -= here;
      }
    }
    tok = c.uin ? c.uin[(size_t)h * c.N + at] : at;
  } else if (j >= s.m_t) return;
  const T* row = X + ((size_t)h * c.N + tok) * D;
  float bsum = 0.f;
#pragma unroll
  for (int q = 0; q < CPL; ++q) {          // the rows are of the I/O type: their copy for the assignment is exact
    const int col = lane + 64 * q;
    const T raw = row[col];
    const float v = Elem<T>::load(&raw);
    const size_t ao = ((size_t)h * c.cap + s.ccount + j) * D + col;
    reinterpret_cast<T*>(c.lp)[ao] = raw;
    c.f32[ao] = v;
    bsum = fmaf(v, v, bsum);
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) bsum += __shfl_xor(bsum, o);
  if (lane == 0) c.bias[(size_t)h * c.cap + s.ccount + j] = -0.5f * bsum;
}

// ------------------------------------------------------------------------------------------
// The late stages of Algorithm 1 in one launch.
// ------------------------------------------------------------------------------------------
// Once every head has few unassigned points left (|U| <= SMALL_NU) and at most SMALL_M centres per
// stage, a stage is six launches of a few microseconds each with next to no work in them, and
// Algorithm 1 may run ten such stages.  Heads are independent, so here ONE workgroup per head runs
// every remaining stage from the loop head to the threshold filter: strided initial sample, `iters`
// assignment passes with the centre update in between, filter and compaction of U, stage
// bookkeeping - the same arithmetic as the separate kernels (same scores, same arg-max, same
// distance, same centre rounding), with the centres, their bias and the member counts in LDS.
//   assignment: as assign_mfma, D[32 centres x 32 points]; a wave takes every NW-th tile of 32 points and
//               runs free of the other waves, with the rows of its next tile in flight;
//   update:     the wave stages its 32 points in LDS and adds S^T[32 dims x 32 centres] += X^T E for
//               them, E the one-hot labels (see stage_pass), into accumulators it keeps for
//               the whole pass; the waves' partial sums are then added in a fixed order, so the result
//               is deterministic;
//   filter:     squared distances of the last pass stay in LDS; U is compacted in ascending order.
constexpr int SMALL_NU = 8192;
constexpr int SMALL_M = 32;

struct SmallStageCfg {
  int N, cap, n_max, m0, m_min, max_stages, u_min, iters;
  const float* tau;               // [1] = tau^2
  int32_t* ulist[2];              // U of stage t is ulist[t & 1]
  bf16raw* cent_lp; float* assign_f32; float* bias;
  int32_t* stage_of;              // may be NULL
  // How the stage before ended, if it has not been closed (both NULL: `st` is that of a stage that has been opened, and its U is in place):
  const int32_t* surv; const int32_t* cnt; int items, cnt_stride;      // its survivors, or
  const float* dist2; TauCfg tc;                                       // (the first stage) its distances, and their sums if tau is to be formed
};

template <int D> struct SmallStage { static constexpr int NW = D == 64 ? 16 : 8; };   // waves (register budget 128 / 256)

template <int D>
__global__ __launch_bounds__(SmallStage<D>::NW * 64) void kstages_small(const bf16raw* __restrict__ X, KState* __restrict__ st,
                                                                       SmallStageCfg cfg) {
  constexpr int LDW = D + 8, KS = D / 16, DT = D / 32, CPL = D / 64;
  constexpr int NW = SmallStage<D>::NW, NT = NW * 64;
  constexpr int SROWB = D * 2 + 16;                  // staged row, padded: the 16-byte pieces of 8 rows fall in 8 bank groups
  constexpr int JPW = SMALL_M / NW;                  // centres a wave finalises
  const int h = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 31, hb = lane >> 5;
  // a wave's staged tile, row-major; between the tile loop and the next pass the partial centre sums of
  // GW waves at a time (rows padded by four floats: the float4 pieces of 8 centres fall in 8 bank groups)
  constexpr int GW = D == 64 ? 8 : 4, PROW = D + 4;
  __shared__ __attribute__((aligned(16))) char xs[NW][32 * SROWB];
  static_assert(sizeof(float) * GW * SMALL_M * PROW <= sizeof(char) * NW * 32 * SROWB, "the partial sums reuse the staging area");
  float* ps = reinterpret_cast<float*>(&xs[0][0]);
  __shared__ __attribute__((aligned(16))) int32_t lab_s[NW][32];
  __shared__ __attribute__((aligned(16))) float fs[SMALL_NU];       // squared distances of the last pass
  __shared__ __attribute__((aligned(16))) bf16raw cs[SMALL_M * LDW];
  __shared__ __attribute__((aligned(16))) float bs[SMALL_M];
  __shared__ int32_t cnt_s[SMALL_M];
  __shared__ int32_t ws[NW];
  __shared__ KState s_st;
  if (tid == 0) s_st = st[h];
  __syncthreads();
  float t2;
  if (cfg.tc.part) {                        // (as keep_count)
    const float t = tau_of<NT>(cfg.tc);
    t2 = t * t;
    if (h == 0 && tid == 0) { cfg.tc.out[0] = t; cfg.tc.out[1] = t2; }
  } else t2 = cfg.tau[1];
  if (!uniform(s_st.active)) return;        // closed before
  // By one thread, with a barrier behind it: a stage ends with `left` points, and the loop goes on or not.  Whatever the loop
  // and its trip counts read of the state is made uniform: the state is in LDS, and with a branch for this thread at the loop's end
  // and another at its head the compiler once let the rest of its wave go on without it, past the barrier.
  auto next_stage = [&](int left) __attribute__((always_inline)) {
    NewState s{left, s_st.ccount + s_st.m_t, 0, s_st.stage + 1, 0, s_st.full, 0};
    loop_head(s, cfg.N, cfg.n_max, cfg.m0, cfg.m_min, cfg.max_stages, cfg.u_min);
    s_st.ucount = s.ucount; s_st.ccount = s.ccount; s_st.m_t = s.m_t; s_st.stage = s.stage;
    s_st.done = s.done; s_st.full = s.full; s_st.active = s.active;
    s_st.stage_offs[s.stage] = s.ccount;
    s_st.u_hist[s.stage] = left;
  };
  // Threshold filter by the distances in LDS: points with d < tau leave U; U stays ascending (as in stage_open).
  auto filter = [&](int n, const int32_t* uin /* NULL: every token */, int32_t* uout, int stage) {
    int run = 0;
    for (int base = 0; base < n; base += 4 * NT) {
      const int p0 = base + 4 * tid;
      bool keep[4]; int tok[4]; int cnt = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int p = p0 + i;
        const bool valid = p < n;
        keep[i] = valid && !(fs[valid ? p : 0] < t2);
        tok[i] = valid ? (uin ? uin[p] : p) : -1;
        cnt += keep[i] ? 1 : 0;
      }
      int incl = cnt;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) { const int v = __shfl_up(incl, o); if (lane >= o) incl += v; }
      __syncthreads();
      if (lane == 63) ws[wave] = incl;
      __syncthreads();
      int before = 0, total = 0;
      for (int w = 0; w < NW; ++w) { const int v = ws[w]; if (w < wave) before += v; total += v; }
      int pos = run + before + incl - cnt;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (keep[i]) uout[pos++] = tok[i];
        else if (tok[i] >= 0 && cfg.stage_of) cfg.stage_of[(size_t)h * cfg.N + tok[i]] = stage;
      }
      run += total;
    }
    return run;
  };
  if (cfg.dist2) {
    const int n0 = uniform(min(s_st.ucount, SMALL_NU)), stage0 = uniform(s_st.stage);
    for (int p = tid; p < n0; p += NT) fs[p] = cfg.dist2[(size_t)h * cfg.N + p];
    __syncthreads();
    const int left = filter(n0, nullptr, cfg.ulist[(stage0 + 1) & 1] + (size_t)h * cfg.N, stage0);
    __syncthreads();
    if (tid == 0) next_stage(left);
    __syncthreads();
  } else if (cfg.surv) {
    // the stage that ended left its survivors: they become U, as stage_open would have moved them
    __shared__ int32_t pre[OPEN_COUNTS + 1];
    const int nb = uniform(min((min(s_st.ucount, cfg.N) + cfg.items - 1) / cfg.items, OPEN_COUNTS));
    const int32_t* cnt = cfg.cnt + (size_t)h * cfg.cnt_stride;
    const int survivors = survivor_prefix(nb, cnt[min(lane, cfg.cnt_stride - 1)], cnt[min(lane + 64, cfg.cnt_stride - 1)], pre);
    int32_t* u = cfg.ulist[(s_st.stage + 1) & 1] + (size_t)h * cfg.N;
    const int total = min(survivors, SMALL_NU);
    for (int p = tid; p < total; p += NT) {
      int at[1] = {p};
      survivors_at(pre, cfg.items, at);
      u[p] = cfg.surv[(size_t)h * cfg.N + at[0]];
    }
    __syncthreads();
    if (tid == 0) next_stage(total);
    __syncthreads();
  }
  // transpose-read addressing of the X^T operand (see stage_pass)
  const int i16 = lane & 15;
  const int vrow = 4 * hb + (i16 >> 2);
  const int gl = 2 * ((lane >> 4) & 1) + ((i16 & 3) >> 1);
  const char* xw = xs[wave] + vrow * SROWB + gl * 16 + 8 * (i16 & 1);

  while (uniform(s_st.active)) {
    const int n = uniform(min(s_st.ucount, SMALL_NU)), m = uniform(min(s_st.m_t, SMALL_M)), row_off = uniform(s_st.ccount), stage = uniform(s_st.stage);
    const int32_t* uin = cfg.ulist[stage & 1] + (size_t)h * cfg.N;
    int32_t* uout = cfg.ulist[(stage + 1) & 1] + (size_t)h * cfg.N;
    const bf16raw* Xh = X + (size_t)h * cfg.N * D;

    // initial centres: strided sample of U (as stage_open); rows past m are zero with a bias that never wins
    if (tid < SMALL_M) cnt_s[tid] = 0;
    for (int j = wave; j < SMALL_M; j += NW) {
      if (j < m) {
        const int tok = uin[sample_at(j, n, m)];
        const bf16raw* row = Xh + (size_t)tok * D;
        float bsum = 0.f;
#pragma unroll
        for (int q = 0; q < CPL; ++q) {
          const int col = lane + 64 * q;
          const bf16raw r = row[col];
          const float img = bf16_to_f32(r);
          cs[j * LDW + col] = r;
          const size_t ao = ((size_t)h * cfg.cap + row_off + j) * D + col;
          cfg.cent_lp[ao] = r;          // an empty cluster keeps this centre to the end of the stage
          cfg.assign_f32[ao] = img;
          bsum = fmaf(img, img, bsum);
        }
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) bsum += __shfl_xor(bsum, o);
        if (lane == 0) { bs[j] = -0.5f * bsum; cfg.bias[(size_t)h * cfg.cap + row_off + j] = -0.5f * bsum; }
      } else {
#pragma unroll
        for (int q = 0; q < CPL; ++q) cs[j * LDW + lane + 64 * q] = 0;
        if (lane == 0) bs[j] = -3.0e38f;
      }
    }
    __syncthreads();

    const int ntiles = (n + 31) >> 5;
    // Rows of a tile: every lane loads its 16-byte pieces of point c.  Both loads are unconditional
    // (positions past the end are clamped to the last point, whose result is then ignored): a load
    // under a branch would make every later wait a wait for all loads in flight.
    auto load_tok = [&](int tile) { return uin[min(tile * 32 + c, n - 1)]; };
    auto load_rows = [&](int tok, bf16x8_t (&x)[KS]) {
      const bf16raw* row = Xh + (size_t)tok * D + hb * 8;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const uint4 raw = *reinterpret_cast<const uint4*>(row + ks * 16);
        x[ks] = *reinterpret_cast<const bf16x8_t*>(&raw);
      }
    };

    for (int it = 0; it < cfg.iters; ++it) {
      const bool update = it < cfg.iters - 1;
      f32x16_t sacc[DT];
#pragma unroll
      for (int b = 0; b < DT; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) sacc[b][v] = 0.f;
      // One tile of 32 points: scores, arg-max, and in an update pass the tile's share of the centre sums.
      auto process = [&](int tile, const bf16x8_t (&x)[KS]) {
        const int p = tile * 32 + c;
        const bool valid = p < n;
        // scores against every centre, arg-max (as assign_mfma)
        f32x16_t acc;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float4 b4 = *reinterpret_cast<const float4*>(&bs[8 * i + 4 * hb]);
          acc[4 * i + 0] = b4.x; acc[4 * i + 1] = b4.y; acc[4 * i + 2] = b4.z; acc[4 * i + 3] = b4.w;
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(&cs[c * LDW + ks * 16 + hb * 8]);
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, x[ks], acc, 0, 0, 0);
        }
        float pk[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) pk[v] = __uint_as_float((__float_as_uint(acc[v]) & 0xFFFFFFF0u) | (uint32_t)(15 - v));
        float best = fmaxf(fmaxf(pk[0], pk[1]), pk[2]);
#pragma unroll
        for (int v = 3; v < 15; v += 2) best = fmaxf(fmaxf(best, pk[v]), pk[v + 1]);
        best = fmaxf(best, pk[15]);
        const int v = 15 - (int)(__float_as_uint(best) & 15u);
        int bidx = 8 * (v >> 2) + 4 * hb + (v & 3);
        float bv = __uint_as_float(__float_as_uint(best) & 0xFFFFFFF0u);
        {
          const float ob = __shfl_xor(bv, 32);
          const int oi = __shfl_xor(bidx, 32);
          if (ob > bv || (ob == bv && oi < bidx)) { bv = ob; bidx = oi; }
        }
        if (!update) {
          // last pass: squared distance to the chosen centre, kept for the filter
          float ss = 0.f;
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) {
            const uint4 raw = *reinterpret_cast<const uint4*>(&x[ks]);
            const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float a = __uint_as_float(w[q] << 16), b = __uint_as_float(w[q] & 0xFFFF0000u);
              ss = fmaf(a, a, ss); ss = fmaf(b, b, ss);
            }
          }
          const float xn2 = ss + __shfl_xor(ss, 32);
          if (hb == 0 && valid) fs[p] = fmaxf(xn2 - 2.f * bv, 0.f);
        } else {
          // update pass: stage the tile (this wave's own LDS, read back by this wave only), count the
          // members, add the tile's share of the centre sums
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) *reinterpret_cast<bf16x8_t*>(xs[wave] + c * SROWB + (ks * 16 + hb * 8) * 2) = x[ks];
          if (hb == 0) {
            lab_s[wave][c] = valid ? bidx : -1;
            if (valid) atomicAdd(&cnt_s[bidx], 1);
          }
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
          for (int g = 0; g < 2; ++g) {
            const int4 l0 = *reinterpret_cast<const int4*>(&lab_s[wave][g * 16 + 4 * hb]);
            const int4 l1 = *reinterpret_cast<const int4*>(&lab_s[wave][g * 16 + 8 + 4 * hb]);
            uint4 e;
            e.x = (l0.x == c ? 0x3F80u : 0u) | (l0.y == c ? 0x3F800000u : 0u);
            e.y = (l0.z == c ? 0x3F80u : 0u) | (l0.w == c ? 0x3F800000u : 0u);
            e.z = (l1.x == c ? 0x3F80u : 0u) | (l1.y == c ? 0x3F800000u : 0u);
            e.w = (l1.z == c ? 0x3F80u : 0u) | (l1.w == c ? 0x3F800000u : 0u);
#pragma unroll
            for (int db = 0; db < DT; ++db) {
              const char* xp = xw + g * 16 * SROWB + db * 64;
              const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)xp);
              const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(xp + 8 * SROWB));
              const s16x4_t both[2] = {lo, hi};
              sacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8_t*>(both),
                                                                 *reinterpret_cast<const bf16x8_t*>(&e), sacc[db], 0, 0, 0);
            }
          }
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();      // the next tile overwrites the staged rows
        }
      };
      if constexpr (NW == 16) {
        // Four waves per SIMD hide the latency of the row loads between them, and 128 registers do not
        // hold a second row buffer: only the token ids run one tile ahead.
        bf16x8_t x0[KS];
        int tk = load_tok(wave);
        for (int tile = wave; tile < ntiles; tile += NW) {
          const int tkn = load_tok(tile + NW);
          load_rows(tk, x0);
          process(tile, x0);
          tk = tkn;
        }
      } else {
        // Software pipeline over this wave's tiles, unrolled twice so that the two row buffers keep
        // their names (a rotating copy would wait for the newest load): rows one tile ahead, token
        // ids two ahead, each token load issued before the row loads of its step.
        bf16x8_t x0[KS], x1[KS];
        int tk = load_tok(wave + NW);
        load_rows(load_tok(wave), x0);
        for (int tile = wave; tile < ntiles; tile += 2 * NW) {
          const int tkn = load_tok(tile + 2 * NW);
          load_rows(tk, x1);
          process(tile, x0);
          if (tile + NW >= ntiles) break;
          tk = load_tok(tile + 3 * NW);
          load_rows(tkn, x0);
          process(tile + NW, x1);
        }
      }
      if (!update) break;
      // The waves' partial sums, GW at a time through LDS, added in wave order by the thread that
      // finalises the element: wave w owns centres w, w+NW, ..., a lane the columns lane, lane+64.
      float tot[JPW][CPL];
#pragma unroll
      for (int a = 0; a < JPW; ++a)
#pragma unroll
        for (int q = 0; q < CPL; ++q) tot[a][q] = 0.f;
#pragma unroll
      for (int grp = 0; grp < NW / GW; ++grp) {
        __syncthreads();                     // the area is free (first group: every wave is out of its tile loop)
        if (wave / GW == grp) {
          // value v of tile db is dim db*32 + 8*(v/4) + 4*hb + v%4 of centre c
#pragma unroll
          for (int db = 0; db < DT; ++db) {
            float* out = ps + ((size_t)((wave % GW) * SMALL_M + c)) * PROW + db * 32 + 4 * hb;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float4 o4 = {sacc[db][4 * i], sacc[db][4 * i + 1], sacc[db][4 * i + 2], sacc[db][4 * i + 3]};
              *reinterpret_cast<float4*>(out + 8 * i) = o4;
            }
          }
        }
        __syncthreads();
#pragma unroll
        for (int a = 0; a < JPW; ++a) {
          const int j = wave + NW * a;
#pragma unroll
          for (int u = 0; u < GW; ++u)
#pragma unroll
            for (int q = 0; q < CPL; ++q) tot[a][q] += ps[((size_t)(u * SMALL_M + j)) * PROW + lane + 64 * q];
        }
      }
      // new centres: member mean, rounded to the I/O type; an empty cluster keeps its centre.  Only the
      // centres of the stage's last assignment are its result: they alone go to global memory.
      const bool last_update = it == cfg.iters - 2;
#pragma unroll
      for (int a = 0; a < JPW; ++a) {
        const int j = wave + NW * a;
        if (j >= m) continue;
        const int nj = cnt_s[j];
        if (lane == 0) cnt_s[j] = 0;
        if (nj > 0) {
          float bsum = 0.f;
#pragma unroll
          for (int q = 0; q < CPL; ++q) {
            const bf16raw r = f32_to_bf16(tot[a][q] / (float)nj);
            const float img = bf16_to_f32(r);
            cs[j * LDW + lane + 64 * q] = r;
            bsum = fmaf(img, img, bsum);
          }
#pragma unroll
          for (int o = 1; o < 64; o <<= 1) bsum += __shfl_xor(bsum, o);
          if (lane == 0) bs[j] = -0.5f * bsum;
        }
        if (last_update) {
#pragma unroll
          for (int q = 0; q < CPL; ++q) {
            const int col = lane + 64 * q;
            const bf16raw r = cs[j * LDW + col];          // written by this lane, now or in an earlier pass
            const size_t ao = ((size_t)h * cfg.cap + row_off + j) * D + col;
            cfg.cent_lp[ao] = r;
            cfg.assign_f32[ao] = bf16_to_f32(r);
          }
          if (lane == 0) cfg.bias[(size_t)h * cfg.cap + row_off + j] = bs[j];
        }
      }
      __syncthreads();
    }

    __syncthreads();
    const int run = filter(n, uin, uout, stage);
    __syncthreads();          // U of the next stage is written, and nobody reads the state any more
    if (tid == 0) next_stage(run);
    __syncthreads();
  }
  if (tid == 0) st[h] = s_st;
}

__global__ void fill_i32(int32_t* p, size_t n, int32_t v) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// ------------------------------------------------------------------------------------------
// compactness (Sec. 3.2.1): MSE_h = mean_n || k_n - c(k_n) ||^2
// ------------------------------------------------------------------------------------------
// One row per group of LPR lanes (16-byte pieces), fp32 inside a row, fp64 across rows; block partials are merged by
// mse_final in a fixed order.  Bound by the trips to a row's label and then its centre: sixteen waves with four rows each in
// flight take a block's 1 024 rows in 4 (d=128, bf16) pairs of trips (four waves, a row at a time: 64; 5 x 9 247 rows 38 us).
constexpr int MSE_ROWS = 1024, MSE_THREADS = 1024;
template <typename T, int D>
__global__ __launch_bounds__(MSE_THREADS) void mse_partial(const T* __restrict__ X, const int32_t* __restrict__ labels,
                                                   const float* __restrict__ cent, int N, int cap, int nblk,
                                                   double* __restrict__ part) {
  constexpr int EV = Vec16<T>::N, LPR = D / EV, RPB = MSE_THREADS / LPR, U = 4;   // rows per block step
  const int h = blockIdx.y, b = blockIdx.x, tid = threadIdx.x;
  const int slot = tid / LPR, cl = tid % LPR;
  double acc = 0.0;
  const int beg = b * MSE_ROWS, end = min(N, beg + MSE_ROWS);
  const int32_t* lab = labels + (size_t)h * N;
  const T* Xh = X + (size_t)h * N * D + cl * EV;
  for (int r0 = beg + slot; r0 < end; r0 += U * RPB) {
    int j[U];
    uint4 raw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = min(r0 + u * RPB, end - 1);
      j[u] = lab[r];
      raw[u] = *reinterpret_cast<const uint4*>(Xh + (size_t)r * D);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float x[EV];
      Vec16<T>::decode(raw[u], x);
      const float* c = cent + ((size_t)h * cap + j[u]) * D + cl * EV;
      float ss = 0.f;
#pragma unroll
      for (int e = 0; e < EV; ++e) { const float df = x[e] - c[e]; ss = fmaf(df, df, ss); }
#pragma unroll
      for (int o = 1; o < LPR; o <<= 1) ss += __shfl_xor(ss, o);
      if (cl == 0 && r0 + u * RPB < end) acc += (double)ss;
    }
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) acc += __shfl_xor(acc, o);
  __shared__ double ws[MSE_THREADS / 64];
  if ((tid & 63) == 0) ws[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < MSE_THREADS / 64; ++w) s += ws[w];
    part[(size_t)h * nblk + b] = s;
  }
}

__global__ __launch_bounds__(256) void mse_final(const double* __restrict__ part, int nblk, int N,
                                                 float* __restrict__ mse) {
  const int h = blockIdx.x, tid = threadIdx.x;
  double s = 0.0;
  for (int i = tid; i < nblk; i += 256) s += part[(size_t)h * nblk + i];
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) s += __shfl_xor(s, o);
  __shared__ double ws[4];
  if ((tid & 63) == 0) ws[tid >> 6] = s;
  __syncthreads();
  if (tid == 0) mse[h] = (float)(((ws[0] + ws[1]) + (ws[2] + ws[3])) / (double)N);
}

// ------------------------------------------------------------------------------------------
// host-side launchers
// ------------------------------------------------------------------------------------------
static inline int chk() { return hipGetLastError() == hipSuccess ? 0 : ADACLUSTER_E_INTERNAL; }

int reduce_part_rows() { return REDUCE_ROWS; }
int pass_sum_centres() { return ACC_MAXM; }
int pass_points(int dtype, bool wide) { return dtype == ADACLUSTER_F32 ? PASS_F32_POINTS : wide ? 2 * PASS_POINTS : PASS_POINTS; }
// fp32 stages by block sums: by width, tokens and first centres of a head alone, never by the number of heads, which must not change
// the bits of any of them.  us of a key clustering, and with update_direct_f32: d=64, 1 x 4 096 points, 16 centres 120 and 141; 30 x 6 000,
// 30 centres 250 and 272; 60 x 1 500, 60 centres 180 and 205; 30 x 16 000, 16 centres 342 and 379; 400 x 1 200, 12 centres 478 and 505; 60 x
// 3 000, 40 centres 324 and 331; d=128, 1 x 4 096, 16 centres 138 and 165; 24 x 4 000 320 and 349; 15 x 6 500, 30 centres 242 and 305;
// 60 x 6 500 670 and 681.  Slower at d=128 in launches of more than some 200 000 points with few centres, where a workgroup a CU
// does not hide its latency: 60 x 4 000, 24 centres 616 and 578, 200 x 1 500, 16 centres 667 and 600.  Past the lines (two tiles of
// centres, 2 MB of sums a head, 40 centres at d=128, which date from passes that formed the centres) they are the faster form
// mostly as well, not by much: 4 x 12 000, d=64, 60 centres 220 and 270, 1 x 12 000, 64 centres 201 and 187; 3 x 4 000, d=128, 50
// centres 180 and 197, 30 x 4 000 428 and 430, 3 x 12 000, 40 centres 218 and 320.
static constexpr int PASS_F32_BYTES = 2 << 20;
int pass_f32_rows(int d, int N, int m0) { return min((long long)(N + PASS_F32_POINTS - 1) / PASS_F32_POINTS * min(m0, PASS_F32_CENTRES), PASS_F32_BYTES / 8ll / d); }
bool pass_f32_fits(int d, int N, int m0) {
  const long long nb = (N + PASS_F32_POINTS - 1) / PASS_F32_POINTS;
  return nb <= STAGE_SUM_BLOCKS && m0 <= (d == 64 ? PASS_F32_CENTRES : 40) && nb * m0 * d * 8 <= PASS_F32_BYTES;
}
// Whether the next pass forms the centres of an fp32 stage, every workgroup for itself, or a launch between the two: the bits are the
// same.  A workgroup's own trips take longer than the launch where a head has more than 512 KB of sums, and what all read together
// counts in launches of many heads.  us of a key clustering, formed by the pass and by a launch: d=64, 1 x 4 096 points, 16 centres
// (262 KB, 8 MB in all) 119 and 125; 10 x 1 500, 12 centres (74 KB, 9 MB) 162 and 175; 1 x 4 096, 32 centres (524 KB, 17 MB) 181 and
// 191; 4 x 4 096, 16 centres (34 MB) 124 and 126; 1 x 6 000, 60 centres (1.4 MB) 218 and 207; 150 x 1 500, 20 centres (221 MB) 350 and
// 319; d=128, 4 x 1 500, 12 centres (147 KB, 7 MB) 154 and 163; 1 x 4 096, 16 centres (524 KB, 17 MB) 131 and 131; 1 x 4 096, 30
// centres (983 KB) 178 and 172; 30 x 1 500, 16 centres (70 MB) 252 and 237; 60 x 6 500, 30 centres (4.8 GB) 1 174 and 670.
bool pass_f32_combines(int d, int heads, int n_bound, int m_bound) {
  const long long nb = (n_bound + PASS_F32_POINTS - 1) / PASS_F32_POINTS, table = nb * m_bound * d * 8;
  return table <= (512 << 10) && table * nb * heads <= 40000000;
}
// Every workgroup of a head reads all of its sums: up to 128 KB they cost less than the launch they save (up to 256 KB the
// same time either way), up to 64 centres or (d=128) 40: each 32 or 16 are another trip (of 3 000 points, d=128, 100 centres at
// first, a call took 540 us without that limit, 477 with launches).  Past some 512 workgroups the chip is full without waves to
// spare for it.
bool combine_fits(int d, int heads, int n_bound, int m_bound) {
  const long long nb = (n_bound + 2 * PASS_POINTS - 1) / (2 * PASS_POINTS);
  return nb * m_bound * d * 4 <= (128 << 10) && m_bound <= (d == 64 ? 64 : 40) && nb * heads <= 512;
}

// Where finalize_centroids forms the centres: twice the points a workgroup are half the sums to write and to read again, once the
// launch still fills the chip (two of these workgroups a CU at d=64).  Key clusterings of 30 x 30 000, d=128, 128 centres 724 ->
// 697 us, of 30 x 17 776, d=64, 555 -> 549; 8 x 17 776 and 12 x 25 500 (280 and 600 workgroups) within 1 % either way.
bool wide_fills(int heads, int n_bound) { return (long long)heads * ((n_bound + 2 * PASS_POINTS - 1) / (2 * PASS_POINTS)) >= 512; }

// Which fp32 assignment: assign_f32 pays for whole tiles (up to 32 centres one, up to 128 four, of which it skips those past
// the count but not their waves), assign_rows for every centre, at little more than the time of a thread's chain of multiply-adds
// while the launch is small.  So the matrix cores take small launches, many centres and, of each tile count, the upper end.
// us, assign_f32 and assign_rows, d=64, 49 152 points: 4 centres 7 and 6, 16 7 and 11, 65 14 and 29; 160 000: 16 17 and 15, 24 17
// and 19, 48 30 and 29, 64 31 and 36, 72 39 and 39; 600 000: 8 49 and 29, 20 49 and 46, 28 49 and 57, 48 102 and 82, 65 130
// and 103, 88 130 and 129, 112 136 and 160.  d=128, 49 152: 4 13 and 10, 12 13 and 16; 60 000 (past three workgroups a CU):
// 16 22 and 18, 24 22 and 24; 393 120: 20 85 and 80, 24 85 and 92; 1 080 000: 4 285 and 113, 32 286 and 281, 36 318 and 307,
// 40 316 and 330, 65 427 and 472.
static bool assign_f32_rows(int d, long long points, int m) {
  const int t = m <= 32 ? 0 : m <= 64 ? 1 : 2;         // one tile, two, three
  struct Line { long long points; int most[3]; };      // from so many points on: most centres for assign_rows
  static constexpr Line d64[] = {{1000000, {26, 64, 96}}, {200000, {21, 60, 84}}, {150000, {17, 49, 67}}, {100000, {12, 35, 0}}, {20000, {4, 0, 0}}};
  static constexpr Line d128[] = {{500000, {32, 36, 0}}, {50000, {20, 0, 0}}, {20000, {6, 0, 0}}};
  auto most = [&](const auto& lines) { for (const Line& l : lines) if (points >= l.points) return l.most[t]; return 0; };
  return m <= (d == 64 ? most(d64) : most(d128));
}

int launch_assign(hipStream_t s, int dtype, int d, int H, int N, int n_bound, int m_bound, int mode, int m_const, int cap,
                  const KState* st, const int32_t* ulist, const void* X, const void* cent_lp, const float* bias,
                  int32_t* labels, float* dist2, int32_t* keep_lab, float* keep_score, const int32_t* seed_lab,
                  const float* seed_score, const float* tau, int32_t* keep_cnt, int keep_stride, double* dist_sum) {
  if ((mode == 3 || keep_lab || seed_lab) && dtype != ADACLUSTER_BF16) return ADACLUSTER_E_INTERNAL;
  AssignCfg c{mode, m_const, N, cap, st, ulist, keep_lab, keep_score, seed_lab, seed_score, tau, keep_cnt, keep_stride, dist_sum};
  if (dtype == ADACLUSTER_BF16) {
    dim3 g((n_bound + ASSIGN_POINTS_LP - 1) / ASSIGN_POINTS_LP, H);
    if (d == 64) assign_mfma<64><<<g, 256, 0, s>>>((const bf16raw*)X, c, (const bf16raw*)cent_lp, bias, labels, dist2);
    else assign_mfma<128><<<g, 256, 0, s>>>((const bf16raw*)X, c, (const bf16raw*)cent_lp, bias, labels, dist2);
  } else {
    dim3 g((n_bound + ASSIGN_POINTS_F32 - 1) / ASSIGN_POINTS_F32, H), gr((n_bound + ROWS_POINTS - 1) / ROWS_POINTS, H);
    const float *x = (const float*)X, *ce = (const float*)cent_lp;
    if (assign_f32_rows(d, (long long)H * n_bound, m_bound)) {
      if (d == 64) assign_rows<64><<<gr, ROWS_POINTS, 0, s>>>(x, c, ce, bias, labels, dist2);
      else assign_rows<128><<<gr, ROWS_POINTS, 0, s>>>(x, c, ce, bias, labels, dist2);
    } else if (m_bound <= 32) {
      if (d == 64) assign_f32<64, 1><<<g, 128, 0, s>>>(x, c, ce, bias, labels, dist2);
      else assign_f32<128, 1><<<g, 128, 0, s>>>(x, c, ce, bias, labels, dist2);
    } else {
      if (d == 64) assign_f32<64, 4><<<g, 512, 0, s>>>(x, c, ce, bias, labels, dist2);
      else assign_f32<128, 4><<<g, 512, 0, s>>>(x, c, ce, bias, labels, dist2);
    }
  }
  return chk();
}

static OpenCfg open_cfg(int N, int cap, const StageRules& r, const KState* in, KState* out, const StageFilter* f, const StageReport& rep) {
  OpenCfg c{};
  c.N = N; c.cap = cap; c.n_max = r.n_max; c.m0 = r.m0; c.m_min = r.m_min; c.max_stages = r.max_stages; c.u_min = r.u_min;
  c.first = f == nullptr;
  c.items = KEEP_ITEMS;
  c.in = in; c.out = out; c.sums = rep.sums; c.report = rep.slot; c.epoch = rep.epoch;
  if (f) {
    c.items = f->items; c.cnt_stride = f->cnt_stride;
    c.dist2 = f->dist2; c.tau = f->tau; c.cnt = f->cnt; c.uin = f->uin; c.uout = f->uout; c.stage_of = f->stage_of; c.stage = f->stage; c.surv = f->surv;
  }
  return c;
}

int launch_stage_pass(hipStream_t s, int dtype, int d, int H, int N, int n_bound, int m_bound, int cap, const KState* st, const int32_t* ulist,
                      const void* X, void* cent_lp, float* cent_f32, float* bias, bool wide, const StageSums* prev, const StageSums* out,
                      const PassEnd* end, const StageOpening* open) {
  AssignCfg c{1, 0, N, cap, st, ulist};
  if (end) {
    c.keep_lab = end->keep_lab; c.keep_score = end->keep_score; c.dist_sum = end->dist_sum;
    c.tau = end->tau; c.keep_cnt = end->keep_cnt; c.keep_stride = end->keep_stride; c.surv = end->surv; c.stage_of = end->stage_of; c.stage = end->stage;
  }
  OpenCfg oc{};
  if (open) {
    oc = open_cfg(N, cap, *open->rules, open->in, open->out, open->filter, *open->report);
    if (open->filter && (!oc.surv || (open->n_before + oc.items - 1) / oc.items > OPEN_COUNTS)) return ADACLUSTER_E_INTERNAL;
  }
  const int pts = pass_points(dtype, wide), nb = (n_bound + pts - 1) / pts;
  const PassSums in = prev ? PassSums{prev->psum, prev->bcnt, m_bound * nb, nb} : PassSums{}, to = out ? PassSums{out->psum, out->bcnt, m_bound * nb, nb} : PassSums{};
  if (m_bound > (dtype == ADACLUSTER_F32 ? PASS_F32_CENTRES : ACC_MAXM) || (prev && (!wide || open)) || !out != (end != nullptr)) return ADACLUSTER_E_INTERNAL;
  const dim3 g(open ? nb + 1 : nb, H);
  float* dist2 = end ? end->dist2 : nullptr;
  if (dtype == ADACLUSTER_F32) {
    auto launch = [&](auto dim) {
      constexpr int DIM = decltype(dim)::value;
      const float* x = (const float*)X;
      float* lp = (float*)cent_lp;
      const uint32_t turns = 0xFFFFFFFFu / nb + 1;
      if (open) stage_pass_f32<DIM, PASS_OPEN><<<g, 512, 0, s>>>(x, c, lp, cent_f32, bias, dist2, nb, turns, in, to, oc);
      else if (prev) stage_pass_f32<DIM, PASS_COMBINE><<<g, 512, 0, s>>>(x, c, lp, cent_f32, bias, dist2, nb, turns, in, to, oc);
      else stage_pass_f32<DIM, PASS_READ><<<g, 512, 0, s>>>(x, c, lp, cent_f32, bias, dist2, nb, turns, in, to, oc);
      return chk();
    };
    return d == 64 ? launch(std::integral_constant<int, 64>{}) : launch(std::integral_constant<int, 128>{});
  }
  const bf16raw* x = (const bf16raw*)X;
  bf16raw* lp = (bf16raw*)cent_lp;
  auto launch = [&](auto dim) {
    constexpr int DIM = decltype(dim)::value;
    if (wide) {
      if (open) stage_pass<DIM, 8, PASS_OPEN><<<g, 512, 0, s>>>(x, c, lp, cent_f32, bias, dist2, in, to, oc);
      else if (prev) stage_pass<DIM, 8, PASS_COMBINE><<<g, 512, 0, s>>>(x, c, lp, cent_f32, bias, dist2, in, to, oc);
      else stage_pass<DIM, 8, PASS_READ><<<g, 512, 0, s>>>(x, c, lp, cent_f32, bias, dist2, in, to, oc);
    } else if (open) stage_pass<DIM, 4, PASS_OPEN><<<g, 256, 0, s>>>(x, c, lp, cent_f32, bias, dist2, in, to, oc);
    else stage_pass<DIM, 4, PASS_READ><<<g, 256, 0, s>>>(x, c, lp, cent_f32, bias, dist2, in, to, oc);
    return chk();
  };
  return d == 64 ? launch(std::integral_constant<int, 64>{}) : launch(std::integral_constant<int, 128>{});
}

int launch_form_centres(hipStream_t s, int d, int H, int n_bound, int m_bound, int cap, const KState* st, const StageSums& sums, void* cent_lp,
                        float* cent_f32, float* bias) {
  const int nb = (n_bound + PASS_F32_POINTS - 1) / PASS_F32_POINTS;
  const PassSums in{sums.psum, sums.bcnt, m_bound * nb, nb};
  const dim3 g((m_bound * (d / 4) + 255) / 256, H);
  if (d == 64) form_centres_f32<64><<<g, 256, 0, s>>>(in, st, cap, (float*)cent_lp, cent_f32, bias);
  else form_centres_f32<128><<<g, 256, 0, s>>>(in, st, cap, (float*)cent_lp, cent_f32, bias);
  return chk();
}

// one-read pass of the query clustering (bf16, at most pass_sum_centres() centres): NP = walks per head
int qpass_walks(int N) { const int sb = (N + 127) / 128; const int subs = (sb + 63) / 64; return (sb + subs - 1) / subs; }
int launch_qpass(hipStream_t s, int d, int H, int N, int m, int cap, int weighted, const void* X, const void* cent_lp,
                 const float* bias, float* psum, int32_t* pcnt) {
  const int sb = (N + 127) / 128, subs = (sb + 63) / 64, NP = (sb + subs - 1) / subs;
  dim3 g(NP, H);
  if (d == 64) qpass_mfma<64><<<g, 256, 0, s>>>((const bf16raw*)X, N, m, cap, subs, weighted, (const bf16raw*)cent_lp, bias, psum, pcnt, NP);
  else qpass_mfma<128><<<g, 256, 0, s>>>((const bf16raw*)X, N, m, cap, subs, weighted, (const bf16raw*)cent_lp, bias, psum, pcnt, NP);
  return chk();
}

int launch_seg_reduce(hipStream_t s, int dtype, int d, int H, int N, int mode, int m_const, int m_bound, int P,
                      const KState* st, int normalize, int want_box, const void* X, const int32_t* perm,
                      const int32_t* offs, int offs_stride, int32_t* poff, int32_t* pcl, float* psum, float* pnorm,
                      float* pmin, float* pmax, int poff_ready) {
  ReduceCfg c{mode, m_const, N, P, m_bound, st, normalize, want_box};
  if (poff_ready == 1) pcl = nullptr;
  dim3 g(P, H);
  if (dtype == ADACLUSTER_BF16) {
    if (d == 64) seg_reduce<bf16raw, 64><<<g, 64, 0, s>>>((const bf16raw*)X, c, perm, offs, offs_stride, poff, pcl, psum, pnorm, pmin, pmax);
    else seg_reduce<bf16raw, 128><<<g, 64, 0, s>>>((const bf16raw*)X, c, perm, offs, offs_stride, poff, pcl, psum, pnorm, pmin, pmax);
  } else if (normalize && !want_box && (long long)P * H <= REDUCE_FEW) {
    if (d == 64) seg_reduce_few<64><<<g, 256, 0, s>>>((const float*)X, c, perm, offs, offs_stride, poff, pcl, psum, pnorm);
    else seg_reduce_few<128><<<g, 256, 0, s>>>((const float*)X, c, perm, offs, offs_stride, poff, pcl, psum, pnorm);
  } else {
    if (d == 64) seg_reduce<float, 64><<<g, 64, 0, s>>>((const float*)X, c, perm, offs, offs_stride, poff, pcl, psum, pnorm, pmin, pmax);
    else seg_reduce<float, 128><<<g, 64, 0, s>>>((const float*)X, c, perm, offs, offs_stride, poff, pcl, psum, pnorm, pmin, pmax);
  }
  return chk();
}

int launch_finalize(hipStream_t s, int dtype, int d, int H, int mode, int m_const, int m_bound, int P, int cap,
                    int master_stride, const KState* st, int spherical, int update_assign, int want_box,
                    const int32_t* offs, int offs_stride, const int32_t* poff, const float* psum, const float* pnorm,
                    const float* pmin, const float* pmax, float* master, void* assign_lp, float* assign_f32,
                    float* bias, float* out_cent, const float* fallback, int32_t* out_sizes,
                    float* out_mean_norm, float* out_bmin, float* out_bmax, const int32_t* blk_cnt, int nb_stride,
                    int blk_points, const StateExport* ex) {
  FinalizeCfg c{mode, m_const, P, m_bound, cap, master_stride, st, spherical, update_assign,
                dtype == ADACLUSTER_BF16, want_box, blk_cnt, nb_stride, blk_points, ex ? *ex : StateExport{}};
  // in final mode every row of the output (up to cap) gets a size, so cover cap rows
  dim3 g(((update_assign ? m_bound : cap) + FIN_ROWS - 1) / FIN_ROWS, H);
  if (d == 64)
    finalize_centroids<64><<<g, 64 * FIN_ROWS, 0, s>>>(c, offs, offs_stride, poff, psum, pnorm, pmin, pmax, master, assign_lp,
                                            assign_f32, bias, out_cent, fallback, out_sizes, out_mean_norm,
                                            out_bmin, out_bmax);
  else
    finalize_centroids<128><<<g, 64 * FIN_ROWS, 0, s>>>(c, offs, offs_stride, poff, psum, pnorm, pmin, pmax, master, assign_lp,
                                             assign_f32, bias, out_cent, fallback, out_sizes, out_mean_norm,
                                             out_bmin, out_bmax);
  return chk();
}

bool direct_update_fits(int dtype, int n_bound, int m_bound) {
  return dtype == ADACLUSTER_F32 && n_bound <= DIRECT_MAX_POINTS && (long long)n_bound * m_bound <= DIRECT_MAX_VISITS;
}
// Up to some 900 workgroups, a round of them, it is the faster form, and past that soon much the slower one, a little later where the
// other form has more rows to sort; the labels that all of them read together count as well.  Key clusterings have fewer centres than
// the bound that the launch is sized for, and the workgroups past them end at once: 2 400.  us of a query clustering, and with the
// sort, the reduction and the combining launch: bf16, d=64, 16 x 1 500 tokens, 8 clusters 50 and 64; 16 x 1 500, 56 clusters 55 and
// 65; 30 x 1 500, 40 64 and 67; 16 x 4 096, 56 (past the second line) 63 and 72; 30 x 400, 20 56 and 56; 30 x 400, 53 67 and 56;
// 24 x 400, 116 86 and 59; d=128, 24 x 400, 37 61 and 68; 30 x 1 500, 40 85 and 82; 24 x 4 096, 25 93 and 93; 30 x 93 clusters of 400
// 98 and 73; fp32, d=64, 16 x 800, 56 83 and 85, 24 x 1 500, 25 96 and 92, 24 x 400, 87 108 and 92.  fp32 at d=128, whose parts a
// wave reads one row pair at a time, gains up to 6 % where query clusters have a few members and loses 7 where they have more: up to
// 24 in the mean (8 x 400, 75 105 and 112; 4 x 1 500, 75 103 and 101; past it 12 x 800, 10 100 and 93).  Keys gain at any size, since
// their boxes cost the three launches more (fp32, d=128, 4 x 4 096, bound 48 96 and 106; 12 x 4 096, 48 122 and 137; fp32, d=64,
// 58 x 312, 48 79 and 85; bf16, d=128, 30 x 1 500, 48 92 and 96; a cold attention call of 27 x 1 224, 80 223 and 229; past the lines
// fp32, d=64, 76 x 722, 48 92 and 87; bf16, d=128, 30 x 2 500, 120 111 and 106).
bool cluster_stats_fits(int dtype, int d, int H, int N, int m_bound, bool keys) {
  const long long groups = (long long)H * m_bound;
  const int most = keys ? 2400 : dtype == ADACLUSTER_BF16 ? 900 + N / (d == 64 ? 3 : 16) : 900;
  return N <= STATS_ITEMS && groups <= most && groups * N <= (dtype == ADACLUSTER_BF16 ? 3000000 : 1500000) &&
         (keys || dtype == ADACLUSTER_BF16 || d == 64 || N <= 24 * m_bound);
}
int launch_cluster_stats(hipStream_t s, int dtype, int d, int H, int N, int mode, int m_const, int m_bound, int cap, const KState* st,
                         int spherical, int want_box, const void* X, const int32_t* labels, int32_t* perm, int32_t* offs, int offs_stride,
                         float* out_cent, const float* fallback, int32_t* out_sizes, float* out_mean_norm, float* out_bmin,
                         float* out_bmax, const StateExport* ex) {
  if (N > STATS_ITEMS) return ADACLUSTER_E_INTERNAL;
  const StatsCfg c{mode, m_const, N, cap, st, spherical, want_box, ex ? *ex : StateExport{}};
  auto launch = [&](auto elem, auto dim) {
    using T = decltype(elem);
    constexpr int DIM = decltype(dim)::value;
    cluster_stats<T, DIM><<<dim3(m_bound, H), STATS_NT, 0, s>>>((const T*)X, c, labels, perm, offs, offs_stride, out_cent, fallback, out_sizes,
                                                                out_mean_norm, out_bmin, out_bmax);
  };
  using std::integral_constant;
  if (dtype == ADACLUSTER_BF16) { if (d == 64) launch(bf16raw{}, integral_constant<int, 64>{}); else launch(bf16raw{}, integral_constant<int, 128>{}); }
  else { if (d == 64) launch(float{}, integral_constant<int, 64>{}); else launch(float{}, integral_constant<int, 128>{}); }
  return chk();
}

int launch_update_direct(hipStream_t s, int d, int H, int N, int m_bound, int cap, int master_stride, const KState* st,
                         const int32_t* labels, const int32_t* ulist, const void* X, float* master, void* assign_lp,
                         float* assign_f32, float* bias) {
  dim3 g(m_bound, H);
  if (d == 64) update_direct_f32<64><<<g, 256, 0, s>>>((const float*)X, N, cap, master_stride, st, labels, ulist, master, (float*)assign_lp, assign_f32, bias);
  else update_direct_f32<128><<<g, 256, 0, s>>>((const float*)X, N, cap, master_stride, st, labels, ulist, master, (float*)assign_lp, assign_f32, bias);
  return chk();
}

int launch_init_centroids(hipStream_t s, int dtype, int d, int H, int N, int m_const, int m_bound,
                          KState* warm, const int32_t* k_count, const int32_t* full_flag, int spherical, int source_master, int cap,
                          int master_stride, const void* X, float* master, void* assign_lp, float* assign_f32,
                          float* bias) {
  dim3 g((m_bound + INIT_ROWS - 1) / INIT_ROWS, H);
  const int lp = dtype == ADACLUSTER_BF16, nt = 64 * INIT_ROWS;
  const WarmStart w{warm, k_count, full_flag};
  if (dtype == ADACLUSTER_BF16) {
    if (d == 64) init_centroids<bf16raw, 64><<<g, nt, 0, s>>>((const bf16raw*)X, N, m_const, w, spherical, source_master, cap, master_stride, lp, master, assign_lp, assign_f32, bias);
    else init_centroids<bf16raw, 128><<<g, nt, 0, s>>>((const bf16raw*)X, N, m_const, w, spherical, source_master, cap, master_stride, lp, master, assign_lp, assign_f32, bias);
  } else {
    if (d == 64) init_centroids<float, 64><<<g, nt, 0, s>>>((const float*)X, N, m_const, w, spherical, source_master, cap, master_stride, lp, master, assign_lp, assign_f32, bias);
    else init_centroids<float, 128><<<g, nt, 0, s>>>((const float*)X, N, m_const, w, spherical, source_master, cap, master_stride, lp, master, assign_lp, assign_f32, bias);
  }
  return chk();
}

int launch_tau_abs(hipStream_t s, float tau_abs, float* tau_out) {
  tau_set<<<1, 64, 0, s>>>(tau_abs, tau_out);
  return chk();
}

int stage_points_per_count(int dtype) { return dtype == ADACLUSTER_BF16 ? ASSIGN_POINTS_LP : ASSIGN_POINTS_F32; }
int launch_keep_count(hipStream_t s, const KState* st, int H, int N, const float* dist2, const double* dist_sum, int sums, float factor,
                      float* tau, int32_t* cnt, int cnt_stride, int32_t* surv, int32_t* stage_of, int* items) {
  const int count = dist_sum ? H * sums : 0;
  TauCfg t{dist_sum, count, (double)H * (double)N, factor, tau};
  if (count > TAU_SUMS) {
    tau_final<<<1, 1024, 0, s>>>(t);
    t.part = nullptr;
  }
  keep_count<<<dim3((N + KEEP_ITEMS - 1) / KEEP_ITEMS, H), 256, 0, s>>>(st, dist2, N, t, tau, cnt, cnt_stride, surv, stage_of);
  *items = KEEP_ITEMS;
  return chk();
}

int launch_stage_open(hipStream_t s, int dtype, int d, int H, int N, int cap, const StageRules& rules, int n_bound, int m_bound,
                      const KState* in, KState* out, const StageFilter* f, const StageReport& report, const void* X, void* assign_lp,
                      float* assign_f32, float* bias) {
  OpenCfg c = open_cfg(N, cap, rules, in, out, f, report);
  c.lp = assign_lp; c.f32 = assign_f32; c.bias = bias;
  if (c.items > KEEP_ITEMS) return ADACLUSTER_E_INTERNAL;
  if (f) c.nblk = (n_bound + c.items - 1) / c.items;
  const dim3 g(c.nblk + (m_bound + 3) / 4 + 1, H);
  if (dtype == ADACLUSTER_BF16) {
    if (d == 64) stage_open<bf16raw, 64><<<g, 256, 0, s>>>((const bf16raw*)X, c);
    else stage_open<bf16raw, 128><<<g, 256, 0, s>>>((const bf16raw*)X, c);
  } else {
    if (d == 64) stage_open<float, 64><<<g, 256, 0, s>>>((const float*)X, c);
    else stage_open<float, 128><<<g, 256, 0, s>>>((const float*)X, c);
  }
  return chk();
}

// Up to how many points a list goes to the one-launch kernel.  A stage there costs a head's workgroup, whatever the number
// of heads, about 11 us and 10.5 ns a point (21 at d=128); in six launches (block sums) it costs 33-37 us and, for every
// head, 0.13-0.17 ns a point (0.27-0.34).  Of one head with 1 500, 2 500, 7 000 points, 30 centres, d=64, a stage takes 29,
// 40, 86 us in the one and 33, 35, 40 in the other form, of 30 heads 30, 41, 88 and 40, 50, 68; d=128 48, 71, 164 and 39, 41,
// 48, and 50, 72, 168 and 52, 65, 109.  With U as it is the lines cross at about 2 048 points (one head, d=64), further out
// the more heads share the launches, and no more from about 64 heads on (72 at d=128): calls of nine stages, 200 heads
// of 3 500 and 8 000 points, d=64, 763 and 1 385 us, in six launches a stage 1 576 and 3 450.  But the points are the bound
// of the stage before, U shrinks, and what follows is in the one launch too: below 3 072 it is taken always (5 heads
// of 9 247 tokens, d=128: the call 612 us, with the line at 1 100 636).  With three launches a stage, as it is now, that call takes
// 446 us, with the line at 2 048, 1 400, 900 and 500 points for any number of heads 449, 449, 465, 465; 1 x 9 000, d=128 264 and 274, 274,
// 275, 291; 3 x 2 587, d=64 135 and 149, 144, 142, 158; 12 x 32 760 and 30 x 17 776 within 1 %.  Calls with a fifth of their heads without
// structure, whose U shrinks slowly, would have it lower: 5 x 9 000, d=64 509 and 466-470, d=128 785 and 593-597; 12 x 9 000 578 and 520, 922
// and 733; 30 x 4 000 500 and 481, 748 and 715, 671; it does not tell the two apart.
int small_stage_points(int d, int heads) {
  const int one = d == 64 ? 2048 : 1024, all = d == 64 ? 64 : 72;
  return heads >= all ? SMALL_NU : min(SMALL_NU, max(3072, one * all / (all - heads)));
}
int small_stage_centres() { return SMALL_M; }
bool small_forms_tau(int H, int sums) { return (long long)H * sums <= TAU_SUMS; }

int launch_kstages_small(hipStream_t s, int d, int H, int N, int cap, const StageRules& r, int iters, KState* st, float* tau,
                         int32_t* ulist0, int32_t* ulist1, const void* X, void* cent_lp, float* assign_f32, float* bias,
                         int32_t* stage_of, const StageFilter* f, int n_before, const double* dist_sum, int sums, float factor) {
  SmallStageCfg cfg{};
  cfg.N = N; cfg.cap = cap; cfg.n_max = r.n_max; cfg.m0 = r.m0; cfg.m_min = r.m_min; cfg.max_stages = r.max_stages;
  cfg.u_min = r.u_min; cfg.iters = iters; cfg.tau = tau; cfg.ulist[0] = ulist0; cfg.ulist[1] = ulist1;
  cfg.cent_lp = (bf16raw*)cent_lp; cfg.assign_f32 = assign_f32; cfg.bias = bias; cfg.stage_of = stage_of;
  if (f && sums > 0) {
    if (n_before > SMALL_NU || !small_forms_tau(H, sums)) return ADACLUSTER_E_INTERNAL;
    cfg.dist2 = f->dist2;
    if (dist_sum) cfg.tc = TauCfg{dist_sum, H * sums, (double)H * (double)N, factor, tau};
  } else if (f) {
    if (!f->surv || (n_before + f->items - 1) / f->items > OPEN_COUNTS) return ADACLUSTER_E_INTERNAL;
    cfg.surv = f->surv; cfg.cnt = f->cnt; cfg.items = f->items; cfg.cnt_stride = f->cnt_stride;
  }
  if (d == 64) kstages_small<64><<<H, SmallStage<64>::NW * 64, 0, s>>>((const bf16raw*)X, st, cfg);
  else kstages_small<128><<<H, SmallStage<128>::NW * 64, 0, s>>>((const bf16raw*)X, st, cfg);
  return chk();
}

int launch_mse(hipStream_t s, int dtype, int d, int H, int N, int cap, const void* X, const int32_t* labels,
               const float* cent, double* part, float* mse) {
  const int nblk = (N + MSE_ROWS - 1) / MSE_ROWS;
  dim3 g(nblk, H);
  if (dtype == ADACLUSTER_BF16) {
    if (d == 64) mse_partial<bf16raw, 64><<<g, MSE_THREADS, 0, s>>>((const bf16raw*)X, labels, cent, N, cap, nblk, part);
    else mse_partial<bf16raw, 128><<<g, MSE_THREADS, 0, s>>>((const bf16raw*)X, labels, cent, N, cap, nblk, part);
  } else {
    if (d == 64) mse_partial<float, 64><<<g, MSE_THREADS, 0, s>>>((const float*)X, labels, cent, N, cap, nblk, part);
    else mse_partial<float, 128><<<g, MSE_THREADS, 0, s>>>((const float*)X, labels, cent, N, cap, nblk, part);
  }
  mse_final<<<H, 256, 0, s>>>(part, nblk, N, mse);
  return chk();
}

int launch_fill_i32(hipStream_t s, int32_t* p, size_t n, int32_t v) {
  if (n == 0) return 0;
  fill_i32<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(p, n, v);
  return chk();
}

}  // namespace adac
