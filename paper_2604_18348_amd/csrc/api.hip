// C ABI of the clustered sparse-attention library: argument checks, workspace layout and the
// order in which the kernels of Algorithm 3 are enqueued.  No device memory is allocated here.
#include "common.h"
#include "launch.h"
#include "stage_report.h"

#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <mutex>

using namespace adac;

// Scratch memory that belongs to the library, for the one entry point that takes no workspace
// (adacluster_compactness_noalloc).  Every GPU the library runs on holds its own copy of the array until
// the process ends.  In host code the name is only a handle for hipGetSymbolAddress: kernels get the
// address that call returns for the current device, never the name.
constexpr size_t STATIC_SCRATCH_DOUBLES = 65536;                 // 512 KiB
static __device__ __align__(256) double scratch[STATIC_SCRATCH_DOUBLES];

namespace {

thread_local char g_err[256] = "";

// Optional stage timing: hipEvents recorded at the stage boundaries of a call.  A stage is timed
// from the event in from[] (default: the previous recorded stage boundary); the fused call runs
// the two clusterings side by side, so both of those are timed from the start of the call.
enum { EV_START = 0, EV_QCLUSTER, EV_KCLUSTER, EV_SELECT, EV_PERMUTE, EV_PLAN, EV_ATTN, EV_KREDUCE, EV_STAGES,
       EV_JOIN = EV_STAGES, EV_KSORT, EV_COUNT };
struct Profiler {
  bool enabled = false;
  bool recorded[EV_COUNT] = {};
  int from[EV_COUNT] = {};
  hipEvent_t ev[EV_COUNT] = {};
} g_prof;

void prof_begin(hipStream_t st) {
  if (!g_prof.enabled) return;
  for (int i = 0; i < EV_COUNT; ++i) { g_prof.recorded[i] = false; g_prof.from[i] = -1; }
  (void)hipEventRecord(g_prof.ev[EV_START], st);
  g_prof.recorded[EV_START] = true;
}
void prof_mark(int which, hipStream_t st, int from = -1) {
  if (!g_prof.enabled) return;
  (void)hipEventRecord(g_prof.ev[which], st);
  g_prof.recorded[which] = true;
  g_prof.from[which] = from;
}

// A second stream per calling thread and device, for work of a call that does not depend on what
// the caller's stream is doing (default priority, like every stream here), and the events that fork
// it from and join it to the caller's stream.  Per thread, so that calls of different host threads
// on one device do not share events.
struct AuxStream {
  bool ready = false;
  hipStream_t s = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
};
thread_local AuxStream g_aux[64];

// Pinned host slots for the per-stage report of Algorithm 1, per thread.  The host polls the last word of a slot, which
// the device writes behind the others: an event would put a barrier between the stage head and the kernels behind it
// (5-8 us a stage).
struct StageReadback {
  bool ready = false;
  int device = -1;
  int epoch = 0;               // of the call that uses the slots: tells its reports from those of the call before
  int32_t* host = nullptr;     // [ADACLUSTER_MAX_STAGES + 2][4], pinned, mapped and coherent
  int32_t* dev = nullptr;      // the same memory as the device sees it
};
thread_local StageReadback t_readback;

StageReadback* stage_readback() {
  StageReadback& r = t_readback;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return nullptr;
  if (r.ready && r.device != dev) {
    (void)hipHostFree(r.host);
    r.ready = false;
  }
  if (!r.ready) {
    r.device = dev;
    const size_t bytes = (ADACLUSTER_MAX_STAGES + 2) * 4 * sizeof(int32_t);
    if (hipHostMalloc((void**)&r.host, bytes, hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) return nullptr;
    memset(r.host, 0, bytes);
    r.epoch = 0;
    if (hipHostGetDevicePointer((void**)&r.dev, r.host, 0) != hipSuccess) { (void)hipHostFree(r.host); return nullptr; }
    r.ready = true;
  }
  r.epoch = r.epoch == INT32_MAX ? 1 : r.epoch + 1;
  return &r;
}

// Waits for the report of stage t.
bool stage_report_landed(const StageReadback& r, int t, hipStream_t st) {
  return report_landed(r.host + 4 * t + 3, r.epoch, st);
}

AuxStream* aux_stream() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  AuxStream& a = g_aux[dev];
  if (!a.ready) {
    if (hipStreamCreateWithFlags(&a.s, hipStreamNonBlocking) != hipSuccess) return nullptr;
    if (hipEventCreateWithFlags(&a.fork, hipEventDisableTiming) != hipSuccess) return nullptr;
    if (hipEventCreateWithFlags(&a.join, hipEventDisableTiming) != hipSuccess) return nullptr;
    a.ready = true;
  }
  return &a;
}

int fail(int code, const char* fmt, ...);

// Device address of `scratch` on the current device, looked up once per device.
std::mutex g_scratch_mu;
double* g_scratch_ptr[64] = {};
double* static_scratch() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
    g_scratch_ptr[dev] = (double*)ptr;
  }
  return g_scratch_ptr[dev];
}

int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

int check_params(const adacluster_params* p) {
  if (!p) return fail(ADACLUSTER_E_BADARG, "params is NULL");
  if (p->H < 1 || p->N < 1) return fail(ADACLUSTER_E_BADSHAPE, "H and N must be >= 1 (H=%d N=%d)", p->H, p->N);
  if (p->H > 65535) return fail(ADACLUSTER_E_BADSHAPE, "H must be <= 65535");
  if (p->d != 64 && p->d != 128) return fail(ADACLUSTER_E_BADSHAPE, "d must be 64 or 128 (d=%d)", p->d);
  if (p->dtype != ADACLUSTER_F32 && p->dtype != ADACLUSTER_BF16) return fail(ADACLUSTER_E_BADDTYPE, "unknown dtype %d", p->dtype);
  if ((long long)p->N * p->d * 4 >= (1ll << 40)) return fail(ADACLUSTER_E_BADSHAPE, "N too large");
  if (p->q_clusters < 1 || p->q_clusters > p->N) return fail(ADACLUSTER_E_BADSHAPE, "q_clusters must be in [1,N]");
  if (p->q_clusters > 4096) return fail(ADACLUSTER_E_BADSHAPE, "q_clusters must be <= 4096");
  if (p->q_iters < 1 || p->k_iters < 1) return fail(ADACLUSTER_E_BADARG, "q_iters and k_iters must be >= 1");
  if (p->q_init_mode != 0 && p->q_init_mode != 1) return fail(ADACLUSTER_E_BADARG, "q_init_mode must be 0 or 1");
  if (p->k_init_mode != 0 && p->k_init_mode != 1) return fail(ADACLUSTER_E_BADARG, "k_init_mode must be 0 or 1");
  if (p->k_m0 < 1 || p->k_m0 > p->N) return fail(ADACLUSTER_E_BADSHAPE, "k_m0 must be in [1,N]");
  if (p->k_m_min < 1 || p->k_m_min > p->k_m0) return fail(ADACLUSTER_E_BADARG, "k_m_min must be in [1,k_m0]");
  if (p->k_max_clusters < 1) return fail(ADACLUSTER_E_BADARG, "k_max_clusters must be >= 1");
  if (p->k_m0 > p->k_max_clusters) return fail(ADACLUSTER_E_BADARG, "k_m0 must not exceed k_max_clusters");
  if ((long long)p->k_max_clusters + p->k_m0 > 7168) return fail(ADACLUSTER_E_BADSHAPE, "k_max_clusters + k_m0 must be <= 7168");
  if (p->k_max_stages < 1 || p->k_max_stages > ADACLUSTER_MAX_STAGES) return fail(ADACLUSTER_E_BADARG, "k_max_stages must be in [1,%d]", ADACLUSTER_MAX_STAGES);
  if (!(p->tau_abs > 0.f) && !(p->tau_factor > 0.f)) return fail(ADACLUSTER_E_BADARG, "tau_abs or tau_factor must be > 0");
  if (!(p->min_unassigned_frac >= 0.f) || p->min_unassigned_frac > 1.f) return fail(ADACLUSTER_E_BADARG, "min_unassigned_frac must be in [0,1]");
  if (p->score_mode < 0 || p->score_mode > 2) return fail(ADACLUSTER_E_BADARG, "unknown score_mode %d", p->score_mode);
  if (p->select_mode < 0 || p->select_mode > 1) return fail(ADACLUSTER_E_BADARG, "unknown select_mode %d", p->select_mode);
  if (p->topk < 1) return fail(ADACLUSTER_E_BADARG, "topk must be >= 1");
  if (!(p->top_p > 0.f) || p->top_p > 1.f) return fail(ADACLUSTER_E_BADARG, "top_p must be in (0,1]");
  if (p->q_no_norm != 0 && p->q_no_norm != 1) return fail(ADACLUSTER_E_BADARG, "q_no_norm must be 0 or 1");
  return 0;
}


inline int capacity(const adacluster_params* p) { return p->k_max_clusters + p->k_m0; }
inline size_t esize(const adacluster_params* p) { return p->dtype == ADACLUSTER_BF16 ? 2 : 4; }
// upper bound of the number of 128-row parts of n rows in m clusters
inline int parts_for(int n, int m) { const int r = reduce_part_rows(); return m + (n + r - 1) / r + 1; }   // every cluster ends in at most one short part

// ---- workspace layout ----------------------------------------------------------------------
struct Layout {
  size_t total = 0;
  size_t take(size_t bytes) { size_t o = total; total += align_up(bytes, 256); return o; }
};

struct WS {
  unsigned char* base;
  KState* kstate; KState* kstate2; int32_t* summary; float* tau;
  void* cent_lp; float* bias;
  int32_t* labels_tmp; float* dist2; int32_t* ulist[2]; int32_t* blockcnt; double* tau_part;
  SortScratch sort; int32_t* perm_tmp; int32_t* offs_tmp; int32_t* poff; int32_t* pcl; int32_t* lab0; float* score0;
  float* psum; float* pnorm; float* pmin; float* pmax; int32_t* bcnt; float* bsum;
  int32_t* perm_q; int32_t* offs_q; int32_t* perm_k; int32_t* offs_k;
  // scratch of the query clustering (its own set: it runs beside the key clustering)
  void* q_cent_lp; float* q_bias; SortScratch q_sort; int32_t* q_poff; float* q_psum; float* q_pnorm;
  float* q_wsum; int32_t* q_wcnt;     // walk sums and counts of the one-read passes of the query clustering
  double* scores;       // [H][Cq][cap] centroid scores between the kernels of the selection step
  int32_t* rng_start; int32_t* rng_pre; int32_t* rng_cnt; int32_t* tiles; int32_t* ntiles;
  int32_t* deal;        // tiles dealt by work (attn_deal_segs)
  int32_t* merge; int32_t* nmerge; float* part_o; float* part_ml;   // cut key lists of the attention step
  int32_t* krow;        // [H][Cq][kstride] every key row of a query cluster's list (see key_row_scale)
  // homes for outputs of the fused call the caller did not ask for
  int32_t* q_labels; float* q_centroids; float* q_assign; int32_t* q_sizes; float* q_mean_norm;
  int32_t* k_labels; float* k_centroids; float* k_assign; float* k_bmin; float* k_bmax;
  int32_t* k_sizes; int32_t* k_count; int32_t* full_flag; int32_t* sel_idx; int32_t* sel_cnt;
  int32_t* one_count;   // [H] constant key-cluster count for the dense plan
  int32_t* sel_keys;    // [H][Cq] keys of every query cluster's list (fused call)
  adacluster_head_stats* stats;   // [H] staging area of adacluster_stats_fetch
};

struct Dims {
  int H, N, d, Cq, cap, capmax, nblk, ncnt, maxtiles, maxr, prow, brow, BM, BMmax;
};

Dims dims_of(const adacluster_params* p) {
  Dims D;
  D.H = p->H; D.N = p->N; D.d = p->d; D.Cq = p->q_clusters; D.cap = capacity(p);
  D.capmax = D.cap > D.Cq ? D.cap : D.Cq;
  D.nblk = (p->N + 1023) / 1024;
  D.ncnt = (p->N + stage_points_per_count(p->dtype) - 1) / stage_points_per_count(p->dtype);
  D.BM = attn_block_rows(p->dtype, p->d, p->N, D.Cq);
  D.BMmax = attn_block_rows_max(p->dtype);
  D.maxtiles = p->N / attn_block_rows_min(p->dtype) + D.Cq + 1 + attn_split_slots();   // (sized for the smaller tile shape)
  D.maxr = D.cap;
  D.prow = p->N / reduce_part_rows() + D.capmax + 34;
  {  // rows of the table of member sums of small stages: blocks x centres, both capped (room for the two tables of stages
     // that combine: those of bf16 have half the blocks, rounded up; those of fp32 hold doubles)
    const int pp = pass_points(ADACLUSTER_BF16, false), nb = (p->N + pp - 1) / pp, mb = p->k_m0 < pass_sum_centres() ? p->k_m0 : pass_sum_centres();
    D.brow = p->dtype == ADACLUSTER_F32 ? 4 * pass_f32_rows(p->d, p->N, p->k_m0) : ((nb < STAGE_SUM_BLOCKS ? nb : STAGE_SUM_BLOCKS) + 1) * mb;
  }
  return D;
}

// K and V stay where they are: the planning step writes, per query cluster, the list of its key rows through the key
// permutation, and the attention kernels load by it (measured against gathering K and V into cluster order first: the
// same attention time, and the gather with its 4 bytes of HBM traffic per input byte gone).  bf16 entries are byte
// offsets inside a head, fp32 entries row numbers.
static int key_row_scale(const adacluster_params* p) { return p->dtype == ADACLUSTER_BF16 ? p->d * 2 : 1; }

size_t layout(const adacluster_params* p, WS* w, unsigned char* base) {
  const Dims D = dims_of(p);
  const size_t H = D.H, N = D.N, d = D.d, es = esize(p);
  Layout L;
#define TAKE(field, type, bytes) { size_t o_ = L.take(bytes); if (w) w->field = (type)(base + o_); }
  TAKE(kstate, KState*, H * sizeof(KState));
  TAKE(kstate2, KState*, H * sizeof(KState));
  TAKE(summary, int32_t*, 64);
  TAKE(tau, float*, 64);
  TAKE(cent_lp, void*, H * D.capmax * d * es);
  TAKE(bias, float*, H * D.capmax * 4);
  TAKE(labels_tmp, int32_t*, H * N * 4);
  TAKE(dist2, float*, H * N * 4);
  TAKE(ulist[0], int32_t*, H * N * 4);
  TAKE(ulist[1], int32_t*, H * N * 4);
  TAKE(blockcnt, int32_t*, H * D.ncnt * 4);
  TAKE(tau_part, double*, H * (D.ncnt > D.nblk ? D.ncnt : D.nblk) * 8);
  TAKE(sort.hist, int32_t*, H * sort_table_ints(D.N, D.capmax) * 4);
  TAKE(sort.lab_a, int32_t*, H * sort_scratch_ints(D.N) * 4);
  TAKE(sort.val_a, int32_t*, H * sort_scratch_ints(D.N) * 4);
  TAKE(sort.lab_b, int32_t*, H * sort_scratch_ints(D.N) * 4);
  TAKE(perm_tmp, int32_t*, H * N * 4);
  TAKE(offs_tmp, int32_t*, H * (size_t)(D.capmax + 1) * 4);
  TAKE(poff, int32_t*, H * (size_t)(D.capmax + 1) * 4);
  TAKE(pcl, int32_t*, H * (size_t)D.prow * 4);
  TAKE(lab0, int32_t*, p->dtype == ADACLUSTER_BF16 ? H * N * 4 : 256);
  TAKE(score0, float*, p->dtype == ADACLUSTER_BF16 ? H * N * 4 : 256);
  TAKE(psum, float*, H * (size_t)D.prow * d * 4);
  TAKE(bcnt, int32_t*, H * (size_t)(p->dtype == ADACLUSTER_F32 ? 2 : 1) * STAGE_SUM_BLOCKS * pass_sum_centres() * 4);      // (bf16: two tables of half the blocks)
  TAKE(bsum, float*, H * (size_t)D.brow * d * 4);
  TAKE(pnorm, float*, H * (size_t)D.prow * 4);
  TAKE(pmin, float*, H * (size_t)D.prow * d * 4);
  TAKE(pmax, float*, H * (size_t)D.prow * d * 4);
  TAKE(q_cent_lp, void*, H * (size_t)D.Cq * d * es);
  TAKE(q_bias, float*, H * (size_t)D.Cq * 4);
  TAKE(q_sort.hist, int32_t*, H * sort_table_ints(D.N, D.Cq) * 4);
  TAKE(q_sort.lab_a, int32_t*, H * sort_scratch_ints(D.N) * 4);
  TAKE(q_sort.val_a, int32_t*, H * sort_scratch_ints(D.N) * 4);
  TAKE(q_sort.lab_b, int32_t*, H * sort_scratch_ints(D.N) * 4);
  TAKE(q_poff, int32_t*, H * (size_t)(D.Cq + 1) * 4);
  TAKE(q_psum, float*, H * (size_t)(N / reduce_part_rows() + D.Cq + 34) * d * 4);
  TAKE(q_pnorm, float*, H * (size_t)(N / reduce_part_rows() + D.Cq + 34) * 4);
  {
    const bool one_read = p->dtype == ADACLUSTER_BF16 && D.Cq <= pass_sum_centres();
    TAKE(q_wsum, float*, one_read ? H * (size_t)D.Cq * qpass_walks(D.N) * d * 4 : 256);
    TAKE(q_wcnt, int32_t*, one_read ? H * (size_t)qpass_walks(D.N) * pass_sum_centres() * 4 : 256);
  }
  TAKE(perm_q, int32_t*, H * N * 4);
  TAKE(offs_q, int32_t*, H * (size_t)(D.Cq + 1) * 4);
  TAKE(perm_k, int32_t*, H * N * 4);
  TAKE(offs_k, int32_t*, H * (size_t)(D.cap + 1) * 4);
  TAKE(scores, double*, H * (size_t)D.Cq * D.cap * 8);
  TAKE(rng_start, int32_t*, H * (size_t)D.Cq * D.maxr * 4);
  TAKE(rng_pre, int32_t*, H * (size_t)D.Cq * (D.maxr + 1) * 4);
  TAKE(rng_cnt, int32_t*, H * (size_t)D.Cq * 4);
  TAKE(tiles, int32_t*, H * (size_t)D.maxtiles * attn_tile_record() * 4);
  TAKE(merge, int32_t*, H * (size_t)attn_split_slots() * 4 * 4);
  TAKE(nmerge, int32_t*, H * 4);
  TAKE(deal, int32_t*, attn_deal_ints(p->dtype, D.d, D.H, D.N, D.Cq, attn_deal_segs(p->dtype, D.d, D.H, D.N, D.Cq, true), attn_most_tiles(p->dtype, D.N, D.Cq, D.BM, D.maxtiles)) * 4);      // (one size for either selection)
  {  // partial results of split key lists: slots of cut lists (bf16), or a row per query and split (fp32; the dense call
     // counts as one cluster, which never makes fewer splits)
    const size_t splits = attn_f32_splits(D.H, D.N, 1);     // (1: the kernel writes the output itself)
    const size_t rows = p->dtype == ADACLUSTER_BF16 ? H * (size_t)attn_split_slots() * D.BMmax : splits > 1 ? H * N * splits : 0;
    TAKE(part_o, float*, rows * d * 4);
    TAKE(part_ml, float*, rows * 2 * 4);
  }
  TAKE(ntiles, int32_t*, H * 4);
  const bool listed = attn_rows_listed(p->dtype, D.d, D.H, D.N, D.Cq);
  TAKE(krow, int32_t*, listed ? H * (size_t)D.Cq * attn_krow_stride(D.N) * 4 : 0);
  if (w && !listed) w->krow = nullptr;
  TAKE(q_labels, int32_t*, H * N * 4);
  TAKE(q_centroids, float*, H * (size_t)D.Cq * d * 4);
  TAKE(q_assign, float*, H * (size_t)D.Cq * d * 4);
  TAKE(q_sizes, int32_t*, H * (size_t)D.Cq * 4);
  TAKE(q_mean_norm, float*, H * (size_t)D.Cq * 4);
  TAKE(k_labels, int32_t*, H * N * 4);
  TAKE(k_centroids, float*, H * (size_t)D.cap * d * 4);
  TAKE(k_assign, float*, H * (size_t)D.cap * d * 4);
  TAKE(k_bmin, float*, H * (size_t)D.cap * d * 4);
  TAKE(k_bmax, float*, H * (size_t)D.cap * d * 4);
  TAKE(k_sizes, int32_t*, H * (size_t)D.cap * 4);
  TAKE(k_count, int32_t*, H * 4);
  TAKE(full_flag, int32_t*, H * 4);
  TAKE(sel_idx, int32_t*, H * (size_t)D.Cq * D.cap * 4);
  TAKE(sel_cnt, int32_t*, H * (size_t)D.Cq * 4);
  TAKE(one_count, int32_t*, H * 4);
  TAKE(sel_keys, int32_t*, (H * (size_t)D.Cq + 1) * 4);
  TAKE(stats, adacluster_head_stats*, H * sizeof(adacluster_head_stats));
#undef TAKE
  if (w) w->base = base;
  return L.total;
}

int check_ws(const adacluster_params* p, void* ws, size_t ws_bytes, WS* w) {
  if (!ws) return fail(ADACLUSTER_E_WORKSPACE, "workspace is NULL");
  if (((uintptr_t)ws) & 255) return fail(ADACLUSTER_E_WORKSPACE, "workspace must be 256-byte aligned");
  const size_t need = layout(p, nullptr, nullptr);
  if (ws_bytes < need) return fail(ADACLUSTER_E_WORKSPACE, "workspace too small: %zu < %zu bytes", ws_bytes, need);
  layout(p, w, (unsigned char*)ws);
  return 0;
}

#define RET_IF(expr) { int rc_ = (expr); if (rc_ != 0) return rc_ == ADACLUSTER_E_INTERNAL ? fail(rc_, "HIP launch failed: %s", hipGetErrorString(hipGetLastError())) : rc_; }
#define PASS_ON(expr) { int rc_ = (expr); if (rc_ != 0) return rc_; }      // (an error that has been reported)

// ---- query clustering ----------------------------------------------------------------------
// passes it0 .. it1 - 1 (the first behind the initial centres)
int run_qcluster(const adacluster_params* p, const WS& w, hipStream_t st, const void* Q, int32_t* q_labels,
                 float* q_centroids, float* q_assign, int32_t* q_sizes, float* q_mean_norm, int it0, int it1) {
  const Dims D = dims_of(p);
  const int P = parts_for(D.N, D.Cq);
  int poff_done = 0;   // set when the sort has already cut the clusters into reduction parts
  const int sph = p->q_no_norm ? 0 : 1;      // by angle on q/|q| (the paper), or Euclidean on raw queries (ablation)
  if (it0 == 0)
    RET_IF(launch_init_centroids(st, p->dtype, D.d, D.H, D.N, D.Cq, D.Cq, nullptr, nullptr, nullptr, sph, p->q_init_mode,
                                 D.Cq, D.Cq, Q, q_centroids, w.q_cent_lp, q_assign, w.q_bias));
  // A pass that only updates the centres reads the queries once: assignment and (normalised) sums in one
  // kernel.  The last pass needs the labels sorted (for the attention step) and exact member statistics, and
  // takes the sort and the segmented reduction.
  const bool one_read = p->dtype == ADACLUSTER_BF16 && D.Cq <= pass_sum_centres();
  for (int it = it0; it < it1; ++it) {
    if (one_read && it < p->q_iters - 1) {
      const int NP = qpass_walks(D.N);
      RET_IF(launch_qpass(st, D.d, D.H, D.N, D.Cq, D.Cq, sph, Q, w.q_cent_lp, w.q_bias, w.q_wsum, w.q_wcnt));
      RET_IF(launch_finalize(st, p->dtype, D.d, D.H, 0, D.Cq, D.Cq, D.Cq * NP, D.Cq, D.Cq, nullptr, sph, 1, 0, nullptr, 0,
                             nullptr, w.q_wsum, w.q_pnorm, nullptr, nullptr, q_centroids, w.q_cent_lp, q_assign, w.q_bias,
                             nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, w.q_wcnt, NP));
      continue;
    }
    RET_IF(launch_assign(st, p->dtype, D.d, D.H, D.N, D.N, D.Cq, 0, D.Cq, D.Cq, nullptr, nullptr, Q, w.q_cent_lp, w.q_bias,
                         q_labels, nullptr));
    if (it == p->q_iters - 1 && cluster_stats_fits(p->dtype, D.d, D.H, D.N, D.Cq, false)) {
      RET_IF(launch_cluster_stats(st, p->dtype, D.d, D.H, D.N, 0, D.Cq, D.Cq, D.Cq, nullptr, sph, 0, Q, q_labels, w.perm_q, w.offs_q, D.Cq + 1,
                                  q_centroids, nullptr, q_sizes, q_mean_norm, nullptr, nullptr, nullptr));
      break;
    }
    RET_IF(launch_sort(st, D.H, D.N, D.N, D.Cq, q_labels, nullptr, nullptr, 0, nullptr, 0, nullptr, 0, w.perm_q,
                       w.offs_q, D.Cq + 1, w.q_sort, w.q_poff, reduce_part_rows(), nullptr, 0, &poff_done));
    RET_IF(launch_seg_reduce(st, p->dtype, D.d, D.H, D.N, 0, D.Cq, D.Cq, P, nullptr, sph, 0, Q, w.perm_q, w.offs_q,
                             D.Cq + 1, w.q_poff, nullptr, w.q_psum, w.q_pnorm, nullptr, nullptr, poff_done));
    const bool last = it == p->q_iters - 1;
    if (!last) {
      RET_IF(launch_finalize(st, p->dtype, D.d, D.H, 0, D.Cq, D.Cq, P, D.Cq, D.Cq, nullptr, sph, 1, 0, w.offs_q,
                             D.Cq + 1, w.q_poff, w.q_psum, w.q_pnorm, nullptr, nullptr, q_centroids, w.q_cent_lp, q_assign, w.q_bias,
                             nullptr, nullptr, nullptr, nullptr, nullptr, nullptr));
    } else {
      RET_IF(launch_finalize(st, p->dtype, D.d, D.H, 0, D.Cq, D.Cq, P, D.Cq, D.Cq, nullptr, sph, 0, 0, w.offs_q,
                             D.Cq + 1, w.q_poff, w.q_psum, w.q_pnorm, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
                             q_centroids, nullptr, q_sizes, q_mean_norm, nullptr, nullptr));
    }
  }
  return 0;
}

// ---- Algorithm 1 ---------------------------------------------------------------------------
// beside(rest): enqueues on another stream what runs beside a cold start: called between two passes of the first stage, and
// (rest: all that is left) before the first wait for the device or at the end of the stages.  A warm start does not call it.
template <typename F>
int run_kcluster(const adacluster_params* p, const WS& w, hipStream_t st, const void* K, int32_t* k_labels,
                 float* k_centroids, float* k_assign, float* k_bmin, float* k_bmax, int32_t* k_sizes,
                 int32_t* k_count, int32_t* full_flag, int32_t* k_stage_offs, int32_t* k_stage_of,
                 float* tau_used, int* kc_bound_out, const F& beside) {
  const Dims D = dims_of(p);
  int kc_bound = 0;   // sum over stages of the largest stage centre count: an upper bound of every |C|
  int pending = 0;                   // the last report (of this stage) may still be in flight when the stage loop ends
  StageReadback* rb = nullptr;
  int poff_done = 0;                 // set when the sort has already cut the clusters into reduction parts
  KState* cur = w.kstate;            // where the state is
  const bool warm = p->k_init_mode == 1;
  if (warm) {
    // warm start: one pseudo-stage over all tokens with the previous centres, count fixed
    cur = w.kstate2;
    if (k_stage_of) RET_IF(launch_fill_i32(st, k_stage_of, (size_t)D.H * D.N, 0));
    RET_IF(launch_init_centroids(st, p->dtype, D.d, D.H, D.N, 0, D.cap, cur, k_count, full_flag, 0, 1, D.cap, D.cap, K,
                                 k_centroids, w.cent_lp, k_assign, w.bias));
    const int Pw = parts_for(D.N, D.cap);
    for (int it = 0; it < p->k_iters; ++it) {
      RET_IF(launch_assign(st, p->dtype, D.d, D.H, D.N, D.N, D.cap, 1, 0, D.cap, cur, nullptr, K, w.cent_lp, w.bias,
                           k_labels, nullptr));
      if (it < p->k_iters - 1 && direct_update_fits(p->dtype, D.N, D.cap)) {
        RET_IF(launch_update_direct(st, D.d, D.H, D.N, D.cap, D.cap, D.cap, cur, k_labels, nullptr, K, k_centroids,
                                    w.cent_lp, k_assign, w.bias));
      } else if (it < p->k_iters - 1) {
        RET_IF(launch_sort(st, D.H, D.N, D.N, D.cap, k_labels, nullptr, nullptr, 0, &cur->m_t, sizeof(KState) / 4,
                           nullptr, 0, w.perm_tmp, w.offs_tmp, D.capmax + 1, w.sort, w.poff, reduce_part_rows(), w.pcl, Pw, &poff_done));
        RET_IF(launch_seg_reduce(st, p->dtype, D.d, D.H, D.N, 1, 0, D.cap, Pw, cur, 0, 0, K, w.perm_tmp,
                                 w.offs_tmp, D.capmax + 1, w.poff, w.pcl, w.psum, w.pnorm, w.pmin, w.pmax, poff_done));
        RET_IF(launch_finalize(st, p->dtype, D.d, D.H, 1, 0, D.cap, Pw, D.cap, D.cap, cur, 0, 1, 0, w.offs_tmp,
                               D.capmax + 1, w.poff, w.psum, w.pnorm, w.pmin, w.pmax, k_centroids, w.cent_lp,
                               k_assign, w.bias, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr));
      }
    }
    kc_bound = D.cap;
  } else {
  const int u_min = (int)floor((double)p->min_unassigned_frac * (double)p->N);
  const bool seeded = p->dtype == ADACLUSTER_BF16;
  double* const dist_sum = p->tau_abs > 0.f ? nullptr : w.tau_part;      // (tau from the distances of the first stage)
  if (k_stage_of) RET_IF(launch_fill_i32(st, k_stage_of, (size_t)D.H * D.N, -1));
  if (p->tau_abs > 0.f) RET_IF(launch_tau_abs(st, p->tau_abs, w.tau));
  // The stage loop has a data-dependent trip count, and grids are sized by what the stage head
  // reports: {active heads, max |U|, max m_t}.  Reading that back before enqueuing the stage
  // would drain the queue once per stage, so the host stays one stage behind: stage t is
  // enqueued with the report of stage t-1 (|U| and m_t never grow, so the older figures are
  // valid bounds; every kernel takes the true counts from the device state), and a stage whose
  // heads all turn out finished runs as empty kernels, once, at the end.  What stage 0 reports the
  // host knows: every head starts alike.
  rb = stage_readback();
  if (!rb) return fail(ADACLUSTER_E_INTERNAL, "stage read-back set-up failed: %s", hipGetErrorString(hipGetLastError()));
  int n_bound = D.N, m_bound = p->k_m0 < D.N ? p->k_m0 : D.N, heads = D.H;
  const StageRules rules{p->k_max_clusters, p->k_m0, p->k_m_min, p->k_max_stages, u_min};
  KState* other = w.kstate2;                       // the stage head reads one and writes the other
  StageFilter filter{};                            // how the stage before ended
  // Stages with few blocks of points and few centres (bf16) update from block sums; they are opened by their own first pass,
  // from the survivors that the stage before left as a list (filter.surv; the first stage: every token).
  const bool f32_sums = p->dtype == ADACLUSTER_F32 && pass_f32_fits(D.d, D.N, m_bound);
  auto sums_fit = [&] {
    if (p->dtype == ADACLUSTER_F32) return f32_sums;
    const int pts = pass_points(p->dtype, false);
    return (n_bound + pts - 1) / pts <= STAGE_SUM_BLOCKS && m_bound <= pass_sum_centres();
  };
  // few points and few centres left in every head: one launch for all stages that follow
  auto small_fits = [&] {
    return p->dtype == ADACLUSTER_BF16 && n_bound <= small_stage_points(D.d, heads) && m_bound <= small_stage_centres();
  };
  int sums_left = 0;                               // distance sums a head that the first stage left to that launch
  for (int t = 0; t <= p->k_max_stages; ++t) {
    const bool pass_opens = t == 0 ? sums_fit() : filter.surv && t < p->k_max_stages;      // (bounds never grow: sums_fit() holds again)
    const int n_before = n_bound;
    // the stage head writes its report straight into the pinned slot (no copy in between)
    const StageReport report{w.summary, t > 0 ? rb->dev + 4 * t : nullptr, rb->epoch};
    if (!pass_opens) {
      if (t > 0) { KState* x = cur; cur = other; other = x; }
      RET_IF(launch_stage_open(st, p->dtype, D.d, D.H, D.N, D.cap, rules, n_bound, m_bound, other, cur, t > 0 ? &filter : nullptr, report,
                               K, w.cent_lp, k_assign, w.bias));
      pending = t;
    }
    if (t > 1) {
      PASS_ON(beside(true));
      if (!stage_report_landed(*rb, t - 1, st))
        return fail(ADACLUSTER_E_INTERNAL, "stage read-back failed: %s", hipGetErrorString(hipGetLastError()));
      const int32_t* summ = rb->host + 4 * (t - 1);
      if (summ[0] == 0) break;                 // stage t-1 had no active head: the loop ended there
      heads = summ[0]; n_bound = summ[1]; m_bound = summ[2];
    }
    if (t > 0) kc_bound += m_bound;
    if (t == p->k_max_stages) break;           // the stage head has just closed every head
    if (t == 1 && !sums_fit()) {
      // Stage 0 removes most points, so its figures (all N points, m_0 centres) are poor bounds for
      // stage 1: unless they still allow the short update (block sums), they would send a few thousand
      // points through the launch chain sized for all of them (label sort, segmented
      // reduction).  Then, once per call, the host waits for the report of the stage it is about to
      // enqueue; the other stream keeps the device busy meanwhile.
      PASS_ON(beside(true));
      if (!stage_report_landed(*rb, 1, st))
        return fail(ADACLUSTER_E_INTERNAL, "stage read-back failed: %s", hipGetErrorString(hipGetLastError()));
      const int32_t* now = rb->host + 4;
      if (now[0] == 0) break;                  // no head needs a second stage
      heads = now[0]; n_bound = now[1]; m_bound = now[2];
    }
    if (t > 0 && small_fits()) {      // (|U|, m_t and the active heads never grow, so the bounds hold for all stages that follow)
      RET_IF(launch_kstages_small(st, D.d, D.H, D.N, D.cap, rules, p->k_iters, cur, w.tau, w.ulist[0], w.ulist[1], K, w.cent_lp, k_assign,
                                  w.bias, k_stage_of, pass_opens ? &filter : nullptr, n_before, dist_sum, sums_left, p->tau_factor));
      kc_bound += m_bound * (p->k_max_stages - t);
      break;
    }
    const int32_t* ul = (t == 0) ? nullptr : w.ulist[t & 1];
    int32_t* ul_next = w.ulist[(t + 1) & 1];
    const int P = parts_for(n_bound, m_bound);
    // A small stage (few blocks of points, few centres) updates its centres from the member sums that a pass leaves per
    // block: no label sort and no segmented reduction in between, and where all of them together are small no launch either.
    const bool block_sums = sums_fit();
    const bool f32 = p->dtype == ADACLUSTER_F32, combine = block_sums && (f32 ? pass_f32_combines : combine_fits)(D.d, heads, n_bound, m_bound);
    const bool wide = combine || (block_sums && !f32 && wide_fills(heads, n_bound));
    const int pts = pass_points(p->dtype, wide), nblk = (n_bound + pts - 1) / pts;
    const StageSums sums[2] = {{w.bsum, w.bcnt}, {w.bsum + (size_t)D.H * m_bound * nblk * D.d * (f32 ? 2 : 1), w.bcnt + (size_t)D.H * nblk * pass_sum_centres()}};
    const int counted = block_sums ? pts : stage_points_per_count(p->dtype);      // points per survivor count and distance sum of the last pass
    // (a stage of block sums has no other use for the array; a single pass would read and write it)
    int32_t* const surv = block_sums && p->k_iters > 1 ? w.labels_tmp : nullptr;
    if (pass_opens && t > 0) { KState* x = cur; cur = other; other = x; }
    const StageOpening opening{&rules, other, cur, t > 0 ? &filter : nullptr, &report, n_before};
    if (pass_opens) pending = t;
    for (int it = 0; it < p->k_iters; ++it) {
      if (t == 0 && it > 0) PASS_ON(beside(false));
      const bool update = it < p->k_iters - 1;
      const bool keep = seeded && t == 0 && !update;
      if (block_sums) {
        const PassEnd end{w.dist2, keep ? w.lab0 : nullptr, keep ? w.score0 : nullptr, t == 0 ? dist_sum : nullptr,
                          w.tau, t > 0 ? w.blockcnt : nullptr, D.ncnt, surv, k_stage_of, t};
        RET_IF(launch_stage_pass(st, p->dtype, D.d, D.H, D.N, n_bound, m_bound, D.cap, cur, ul, K, w.cent_lp, k_assign, w.bias, wide,
                                 combine && it > 0 ? &sums[(it - 1) & 1] : nullptr, update ? &sums[combine ? it & 1 : 0] : nullptr,
                                 update ? nullptr : &end, pass_opens && it == 0 ? &opening : nullptr));
        if (update && !combine && f32) {
          RET_IF(launch_form_centres(st, D.d, D.H, n_bound, m_bound, D.cap, cur, sums[0], w.cent_lp, k_assign, w.bias));
        } else if (update && !combine) {
          RET_IF(launch_finalize(st, p->dtype, D.d, D.H, 1, 0, m_bound, m_bound * nblk, D.cap, 0, cur, 0, 1, 0,
                                 nullptr, 0, nullptr, w.bsum, w.pnorm, w.pmin, w.pmax, nullptr, w.cent_lp,
                                 k_assign, w.bias, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, w.bcnt, nblk, pts));
        }
        continue;
      }
      // (the last pass of stage 0 runs over all points against the first-stage centres as they will stay:
      // it keeps a copy of its labels and best scores, which the final pass starts from)
      RET_IF(launch_assign(st, p->dtype, D.d, D.H, D.N, n_bound, m_bound, 1, 0, D.cap, cur, ul, K, w.cent_lp, w.bias,
                           w.labels_tmp, update ? nullptr : w.dist2, keep ? w.lab0 : nullptr,
                           keep ? w.score0 : nullptr, nullptr, nullptr, w.tau,
                           !update && t > 0 ? w.blockcnt : nullptr, D.ncnt, !update && t == 0 ? dist_sum : nullptr));
      if (update && direct_update_fits(p->dtype, n_bound, m_bound)) {
        // few points (fp32): every centre gathers its members from the label list itself, one launch
        RET_IF(launch_update_direct(st, D.d, D.H, D.N, m_bound, D.cap, 0, cur, w.labels_tmp, ul, K, nullptr,
                                    w.cent_lp, k_assign, w.bias));
      } else if (update) {
        RET_IF(launch_sort(st, D.H, D.N, n_bound, m_bound, w.labels_tmp, ul, &cur->ucount,
                           sizeof(KState) / 4, &cur->m_t, sizeof(KState) / 4, &cur->active,
                           sizeof(KState) / 4, w.perm_tmp, w.offs_tmp, D.capmax + 1, w.sort, w.poff, reduce_part_rows(), w.pcl, P, &poff_done));
        RET_IF(launch_seg_reduce(st, p->dtype, D.d, D.H, D.N, 1, 0, m_bound, P, cur, 0, 0, K, w.perm_tmp,
                                 w.offs_tmp, D.capmax + 1, w.poff, w.pcl, w.psum, w.pnorm, w.pmin, w.pmax, poff_done));
        RET_IF(launch_finalize(st, p->dtype, D.d, D.H, 1, 0, m_bound, P, D.cap, 0, cur, 0, 1, 0,
                               w.offs_tmp, D.capmax + 1, w.poff, w.psum, w.pnorm, w.pmin, w.pmax, nullptr, w.cent_lp,
                               k_assign, w.bias, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr));
      }
    }
    filter = StageFilter{w.dist2, w.tau, w.blockcnt, D.ncnt, counted, ul, ul_next, k_stage_of, t, surv};
    if (t == 0) {
      const int sums = (D.N + counted - 1) / counted;
      if (surv && p->k_max_stages > 1 && small_fits() && small_forms_tau(D.H, sums)) sums_left = sums;
      else RET_IF(launch_keep_count(st, cur, D.H, D.N, w.dist2, dist_sum, sums, p->tau_factor, w.tau, w.blockcnt, D.ncnt, surv, k_stage_of, &filter.items));
    }
  }
  PASS_ON(beside(true));
  kc_bound = kc_bound < D.cap ? kc_bound : D.cap;
  // last step of Algorithm 1: nearest centre among all stage centres, then member statistics.  bf16: the
  // nearest first-stage centre of every point is known from stage 0, so only the later stages' centres are visited.
  if (seeded)
    RET_IF(launch_assign(st, p->dtype, D.d, D.H, D.N, D.N, kc_bound, 3, 0, D.cap, cur, nullptr, K, w.cent_lp, w.bias,
                         k_labels, nullptr, nullptr, nullptr, w.lab0, w.score0))
  else
    RET_IF(launch_assign(st, p->dtype, D.d, D.H, D.N, D.N, kc_bound, 2, 0, D.cap, cur, nullptr, K, w.cent_lp, w.bias,
                         k_labels, nullptr));
  }
  const int want_box = (k_bmin && k_bmax) ? 1 : 0;
  if (kc_bound_out) *kc_bound_out = kc_bound;
  const StateExport ex{w.kstate, k_count, full_flag, k_stage_offs, w.tau, warm ? nullptr : tau_used};
  if (cluster_stats_fits(p->dtype, D.d, D.H, D.N, kc_bound, true)) {
    prof_mark(EV_KSORT, st);
    RET_IF(launch_cluster_stats(st, p->dtype, D.d, D.H, D.N, warm ? 1 : 2, 0, kc_bound, D.cap, cur, 0, want_box, K, k_labels, w.perm_k, w.offs_k,
                                D.cap + 1, k_centroids, k_assign, k_sizes, nullptr, k_bmin, k_bmax, &ex));
    prof_mark(EV_KREDUCE, st, EV_KSORT);
  } else {
    const int P = parts_for(D.N, kc_bound);
    RET_IF(launch_sort(st, D.H, D.N, D.N, kc_bound, k_labels, nullptr, nullptr, 0, warm ? &cur->m_t : &cur->ccount, sizeof(KState) / 4,
                       nullptr, 0, w.perm_k, w.offs_k, D.cap + 1, w.sort, w.poff, reduce_part_rows(), w.pcl, P, &poff_done));
    prof_mark(EV_KSORT, st);
    RET_IF(launch_seg_reduce(st, p->dtype, D.d, D.H, D.N, warm ? 1 : 2, 0, kc_bound, P, cur, 0, want_box, K, w.perm_k, w.offs_k,
                             D.cap + 1, w.poff, w.pcl, w.psum, w.pnorm, w.pmin, w.pmax, poff_done));
    prof_mark(EV_KREDUCE, st, EV_KSORT);
    RET_IF(launch_finalize(st, p->dtype, D.d, D.H, warm ? 1 : 2, 0, kc_bound, P, D.cap, D.cap, cur, 0, 0, want_box, w.offs_k,
                           D.cap + 1, w.poff, w.psum, w.pnorm, w.pmin, w.pmax, nullptr, nullptr, nullptr, nullptr, k_centroids,
                           k_assign, k_sizes, nullptr, k_bmin, k_bmax, nullptr, 0, 0, &ex));
  }
  // the pinned report slots are reused by the next call of this thread: let the last report land
  // (its kernel was queued ahead of everything above, so this does not drain the stream)
  if (pending && !stage_report_landed(*rb, pending, st))
    return fail(ADACLUSTER_E_INTERNAL, "stage read-back failed: %s", hipGetErrorString(hipGetLastError()));
  return 0;
}

// ---- attention over selected clusters, given both sorts ---------------------------------------
// range lists, row offsets and query tiles from the selection, then the attention kernel
int run_plan_attention(const adacluster_params* p, const WS& w, hipStream_t st, const void* Q, void* O,
                       const int32_t* k_count, const int32_t* sel_idx, const int32_t* sel_cnt, const int32_t* sel_keys, int prof_from,
                       const void* K, const void* V) {
  const Dims D = dims_of(p);
  const float scale = p->softmax_scale > 0.f ? p->softmax_scale : 1.0f / sqrtf((float)D.d);
  const int segs = attn_deal_segs(p->dtype, D.d, D.H, D.N, D.Cq, p->select_mode == ADACLUSTER_SELECT_TOPP), most = attn_most_tiles(p->dtype, D.N, D.Cq, D.BM, D.maxtiles);
  RET_IF(launch_plan_sparse(st, p->dtype, D.d, D.H, D.Cq, D.cap, D.maxr, D.maxtiles, D.BM, w.offs_q, D.Cq + 1, w.offs_k,
                            D.cap + 1, k_count, sel_idx, sel_cnt, w.rng_start, w.rng_pre, w.rng_cnt, w.tiles, w.ntiles,
                            w.merge, w.nmerge, key_row_scale(p), w.krow, attn_krow_stride(D.N), w.perm_k, D.N, sel_keys, segs, most, w.deal, w.sel_keys + (size_t)D.H * D.Cq));
  prof_mark(EV_PLAN, st, prof_from);
  RET_IF(launch_attention(st, p->dtype, D.d, D.H, D.N, D.Cq, D.BM, most, D.maxtiles, scale, Q, K, V, O, w.perm_q,
                          w.tiles, w.ntiles, w.part_o, w.part_ml, w.merge, w.nmerge,
                          w.krow, attn_krow_stride(D.N), w.rng_start, w.rng_pre, w.rng_cnt, D.maxr, w.perm_k, segs, w.deal));
  prof_mark(EV_ATTN, st);
  return 0;
}

}  // namespace

// ---------------------------------------------------------------------------------------------
extern "C" {

int adacluster_centroid_capacity(const adacluster_params* p) {
  int rc = check_params(p);
  if (rc) return rc;
  return capacity(p);
}

int adacluster_workspace_bytes(const adacluster_params* p, size_t* bytes) {
  int rc = check_params(p);
  if (rc) return rc;
  if (!bytes) return fail(ADACLUSTER_E_BADARG, "bytes is NULL");
  *bytes = layout(p, nullptr, nullptr);
  return 0;
}

int adacluster_last_error(char* buf, size_t buf_bytes) {
  if (!buf || buf_bytes == 0) return ADACLUSTER_E_BADARG;
  strncpy(buf, g_err, buf_bytes - 1);
  buf[buf_bytes - 1] = 0;
  return 0;
}

int adacluster_qcluster(const adacluster_params* p, const void* Q, int32_t* q_labels, float* q_centroids,
                        float* q_assign_centroids, int32_t* q_sizes, float* q_mean_norm, void* ws,
                        size_t ws_bytes, void* stream) {
  int rc = check_params(p);
  if (rc) return rc;
  if (!Q || !q_labels || !q_centroids || !q_assign_centroids || !q_sizes || !q_mean_norm)
    return fail(ADACLUSTER_E_BADARG, "qcluster: NULL tensor pointer");
  WS w;
  if ((rc = check_ws(p, ws, ws_bytes, &w))) return rc;
  prof_begin((hipStream_t)stream);
  rc = run_qcluster(p, w, (hipStream_t)stream, Q, q_labels, q_centroids, q_assign_centroids, q_sizes, q_mean_norm, 0, p->q_iters);
  prof_mark(EV_QCLUSTER, (hipStream_t)stream, EV_START);
  return rc;
}

int adacluster_kcluster(const adacluster_params* p, const void* K, int32_t* k_labels, float* k_centroids,
                        float* k_assign_centroids, float* k_box_min, float* k_box_max, int32_t* k_sizes,
                        int32_t* k_count, int32_t* full_flag, int32_t* k_stage_offs, int32_t* k_stage_of,
                        float* tau_used, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_params(p);
  if (rc) return rc;
  if (!K || !k_labels || !k_centroids || !k_assign_centroids || !k_sizes || !k_count || !full_flag || !tau_used)
    return fail(ADACLUSTER_E_BADARG, "kcluster: NULL tensor pointer");
  if ((k_box_min == nullptr) != (k_box_max == nullptr))
    return fail(ADACLUSTER_E_BADARG, "kcluster: pass both boxes or neither");
  WS w;
  if ((rc = check_ws(p, ws, ws_bytes, &w))) return rc;
  prof_begin((hipStream_t)stream);
  rc = run_kcluster(p, w, (hipStream_t)stream, K, k_labels, k_centroids, k_assign_centroids, k_box_min, k_box_max,
                    k_sizes, k_count, full_flag, k_stage_offs, k_stage_of, tau_used, nullptr, [](bool) { return 0; });
  prof_mark(EV_KCLUSTER, (hipStream_t)stream, EV_START);
  return rc;
}

int adacluster_compactness(const adacluster_params* p, const void* K, const int32_t* k_labels,
                           const float* k_centroids, float* k_mse, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_params(p);
  if (rc) return rc;
  if (!K || !k_labels || !k_centroids || !k_mse) return fail(ADACLUSTER_E_BADARG, "compactness: NULL pointer");
  WS w;
  if ((rc = check_ws(p, ws, ws_bytes, &w))) return rc;
  RET_IF(launch_mse((hipStream_t)stream, p->dtype, p->d, p->H, p->N, capacity(p), K, k_labels, k_centroids, w.tau_part,
                    k_mse));
  return 0;
}

int adacluster_compactness_noalloc(const adacluster_params* p, const void* K, const int32_t* k_labels,
                                   const float* k_centroids, float* k_mse, void* stream) {
  int rc = check_params(p);
  if (rc) return rc;
  if (!K || !k_labels || !k_centroids || !k_mse) return fail(ADACLUSTER_E_BADARG, "compactness_noalloc: NULL pointer");
  const size_t need = (size_t)p->H * (size_t)((p->N + 1023) / 1024);   // one partial sum per head and 1024 rows
  if (need > STATIC_SCRATCH_DOUBLES)
    return fail(ADACLUSTER_E_UNSUPPORTED, "compactness_noalloc: H * ceil(N/1024) = %zu exceeds the %zu partial sums of the "
                "library's scratch array; use adacluster_compactness with a workspace", need, STATIC_SCRATCH_DOUBLES);
  double* part = static_scratch();
  if (!part) return fail(ADACLUSTER_E_INTERNAL, "compactness_noalloc: hipGetSymbolAddress failed: %s", hipGetErrorString(hipGetLastError()));
  // every partial sum the second kernel reads is written by the first: nothing has to start at zero
  RET_IF(launch_mse((hipStream_t)stream, p->dtype, p->d, p->H, p->N, capacity(p), K, k_labels, k_centroids, part, k_mse));
  return 0;
}

int adacluster_quest_scores(int32_t H, int32_t Lq, int32_t Lk, int32_t d, int32_t dtype, int32_t form, int32_t clamp,
                            const void* Q, const void* R_pos, const void* R_neg, float* S, void* stream) {
  if (H < 1 || Lq < 1 || Lk < 1) return fail(ADACLUSTER_E_BADSHAPE, "quest_scores: H, Lq and Lk must be >= 1");
  if (H > 65535) return fail(ADACLUSTER_E_BADSHAPE, "quest_scores: H must be <= 65535");
  if (d != 64 && d != 128) return fail(ADACLUSTER_E_BADSHAPE, "quest_scores: d must be 64 or 128 (d=%d)", d);
  if (dtype != ADACLUSTER_F32 && dtype != ADACLUSTER_BF16) return fail(ADACLUSTER_E_BADDTYPE, "quest_scores: unknown dtype %d", dtype);
  if (form != ADACLUSTER_QUEST_ALU && form != ADACLUSTER_QUEST_MFMA) return fail(ADACLUSTER_E_BADARG, "quest_scores: unknown form %d", form);
  if (form == ADACLUSTER_QUEST_MFMA && dtype != ADACLUSTER_BF16)
    return fail(ADACLUSTER_E_UNSUPPORTED, "quest_scores: the matrix-core form takes bf16 inputs");
  if ((long long)Lq * Lk >= (1ll << 40) || (long long)Lq * d >= (1ll << 40) || (long long)Lk * d >= (1ll << 40))
    return fail(ADACLUSTER_E_BADSHAPE, "quest_scores: problem too large");
  if ((Lq + 63) / 64 > 2147483647 / 2 || (Lk + 63) / 64 > 65535) return fail(ADACLUSTER_E_BADSHAPE, "quest_scores: Lk must be <= 4194240");
  if (!Q || !R_pos || !R_neg || !S) return fail(ADACLUSTER_E_BADARG, "quest_scores: NULL pointer");
  RET_IF(launch_quest_scores((hipStream_t)stream, dtype, form, clamp ? 1 : 0, H, Lq, Lk, d, Q, R_pos, R_neg, S));
  return 0;
}

int adacluster_select(const adacluster_params* p, const float* q_centroids, const float* q_mean_norm,
                      const float* k_centroids, const float* k_box_min, const float* k_box_max,
                      const int32_t* k_sizes, const int32_t* k_count, const int32_t* full_flag,
                      int32_t* sel_idx, int32_t* sel_cnt, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_params(p);
  if (rc) return rc;
  if (!q_centroids || !q_mean_norm || !k_centroids || !k_sizes || !k_count || !full_flag || !sel_idx || !sel_cnt)
    return fail(ADACLUSTER_E_BADARG, "select: NULL tensor pointer");
  if (p->score_mode == ADACLUSTER_SCORE_BOX && (!k_box_min || !k_box_max))
    return fail(ADACLUSTER_E_BADARG, "select: BOX scores need k_box_min and k_box_max");
  WS w;
  if ((rc = check_ws(p, ws, ws_bytes, &w))) return rc;
  const float scale = p->softmax_scale > 0.f ? p->softmax_scale : 1.0f / sqrtf((float)p->d);
  RET_IF(launch_select((hipStream_t)stream, p->H, p->q_clusters, capacity(p), p->d, p->score_mode, p->select_mode,
                       p->topk, p->top_p, scale, q_centroids, q_mean_norm, k_centroids, k_box_min, k_box_max, k_sizes,
                       k_count, full_flag, sel_idx, sel_cnt, capacity(p), w.scores, nullptr));
  return 0;
}

int adacluster_sparse_attn(const adacluster_params* p, const void* Q, const void* K, const void* V,
                           const int32_t* q_labels, const int32_t* k_labels, const int32_t* k_count,
                           const int32_t* sel_idx, const int32_t* sel_cnt, void* O, void* ws, size_t ws_bytes,
                           void* stream) {
  int rc = check_params(p);
  if (rc) return rc;
  if (!Q || !K || !V || !q_labels || !k_labels || !k_count || !sel_idx || !sel_cnt || !O)
    return fail(ADACLUSTER_E_BADARG, "sparse_attn: NULL tensor pointer");
  WS w;
  if ((rc = check_ws(p, ws, ws_bytes, &w))) return rc;
  const Dims D = dims_of(p);
  hipStream_t st = (hipStream_t)stream;
  prof_begin(st);
  RET_IF(launch_sort(st, D.H, D.N, D.N, D.Cq, q_labels, nullptr, nullptr, 0, nullptr, 0, nullptr, 0, w.perm_q, w.offs_q,
                     D.Cq + 1, w.sort, nullptr, 0, nullptr, 0, nullptr, 1));
  RET_IF(launch_sort(st, D.H, D.N, D.N, D.cap, k_labels, nullptr, nullptr, 0, k_count, 1, nullptr, 0, w.perm_k, w.offs_k,
                     D.cap + 1, w.sort, nullptr, 0, nullptr, 0, nullptr, 1));
  prof_mark(EV_SELECT, st);   // (time of the two label sorts when called stand-alone)
  return run_plan_attention(p, w, st, Q, O, k_count, sel_idx, sel_cnt, nullptr, -1, K, V);
}

int adacluster_attn(const adacluster_params* p, const void* Q, const void* K, const void* V, void* O,
                    const adacluster_outputs* outs, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_params(p);
  if (rc) return rc;
  if (!Q || !K || !V || !O) return fail(ADACLUSTER_E_BADARG, "attn: NULL tensor pointer");
  WS w;
  if ((rc = check_ws(p, ws, ws_bytes, &w))) return rc;
  adacluster_outputs o;
  memset(&o, 0, sizeof(o));
  if (outs) o = *outs;
  if ((o.k_box_min == nullptr) != (o.k_box_max == nullptr))
    return fail(ADACLUSTER_E_BADARG, "attn: pass both boxes or neither");
  const bool need_box = p->score_mode == ADACLUSTER_SCORE_BOX;
#define PICK(f, home) auto f = o.f ? o.f : home
  PICK(q_labels, w.q_labels); PICK(q_centroids, w.q_centroids); PICK(q_assign_centroids, w.q_assign);
  PICK(q_sizes, w.q_sizes); PICK(q_mean_norm, w.q_mean_norm);
  PICK(k_labels, w.k_labels); PICK(k_centroids, w.k_centroids); PICK(k_assign_centroids, w.k_assign);
  PICK(k_sizes, w.k_sizes); PICK(k_count, w.k_count); PICK(full_flag, w.full_flag);
  PICK(sel_idx, w.sel_idx); PICK(sel_cnt, w.sel_cnt);
#undef PICK
  float* k_bmin = o.k_box_min ? o.k_box_min : (need_box ? w.k_bmin : nullptr);
  float* k_bmax = o.k_box_max ? o.k_box_max : (need_box ? w.k_bmax : nullptr);
  float* tau_used = o.tau_used ? o.tau_used : w.tau + 2;
  hipStream_t st = (hipStream_t)stream;
  if (p->q_init_mode == 1 && !o.q_centroids)
    return fail(ADACLUSTER_E_BADARG, "attn: q_init_mode 1 needs outs->q_centroids");
  if (p->k_init_mode == 1 && (!o.k_centroids || !o.k_count || !o.full_flag))
    return fail(ADACLUSTER_E_BADARG, "attn: k_init_mode 1 needs outs->k_centroids, k_count and full_flag");
  // The two clusterings do not depend on each other and both are chains of small kernels: the
  // query clustering goes to a second stream, forked from and joined back to the caller's.
  AuxStream* aux = aux_stream();
  if (!aux) return fail(ADACLUSTER_E_INTERNAL, "could not create the second stream: %s", hipGetErrorString(hipGetLastError()));
  prof_begin(st);
  if (hipEventRecord(aux->fork, st) != hipSuccess || hipStreamWaitEvent(aux->s, aux->fork, 0) != hipSuccess)
    return fail(ADACLUSTER_E_INTERNAL, "stream fork failed: %s", hipGetErrorString(hipGetLastError()));
  // From here on work may sit on the second stream.  No error leaves this function with that work still
  // running: where the event join itself fails (or an error comes after the join of the first fork), the
  // host waits for the second stream before it reports the error.
  auto drained = [&](int code) { (void)hipStreamSynchronize(aux->s); return code; };
  hipStream_t qs = aux->s;      // (measured: run in front of Algorithm 1 on the caller's stream instead, every configuration is 1-6 % slower)
  // Algorithm 1 is the longer chain.  Where it waits for a report, it goes first, and the query clustering is enqueued while the
  // host would only wait; its nine launches ahead of Algorithm 1 kept the device waiting (4 096 fp32 tokens 240 -> 221 us;
  // 32 760 tokens, a call alone, 863 -> 840).  Where no report is waited for before the end (a warm start, or one launch for
  // everything after the first stage) it stays first: 1 500 tokens, call after call, 146 us, 157 in turn.
  // With more query clusters than a pass sums itself, every pass of theirs is a chain of four to six launches, and together they
  // can be the longer chain: a pass of either side in turn, until the host waits.  Algorithm 1 first, in turn and query clustering
  // first, us for calls alone: 4 x 4 096 tokens, d=64, 256 query clusters 227, 209, 209; 1 x 4 096 fp32, 256 252, 229, 218; 5 x
  // 9 247, d=128, 512 412, 392, 392; 168 shapes from 1 500 to 75 600 tokens, 129 to 1 024 query clusters: in turn 0.96 of Algorithm 1
  // first, call after call 0.99.
  const bool q_first = p->k_init_mode == 1 || (p->dtype == ADACLUSTER_BF16 && p->N <= small_stage_points(p->d, p->H) && p->k_m0 <= small_stage_centres());
  const bool in_turn = p->q_clusters > pass_sum_centres();
  bool joinable = false;
  int q_it = 0;                 // passes of the query clustering that are enqueued
  auto queries = [&](bool rest) {
    if (q_it >= p->q_iters || (!rest && !in_turn)) return 0;
    const int from = q_it;
    q_it = rest ? p->q_iters : q_it + 1;
    const int r = run_qcluster(p, w, qs, Q, q_labels, q_centroids, q_assign_centroids, q_sizes, q_mean_norm, from, q_it);
    if (r) q_it = p->q_iters;
    if (q_it < p->q_iters) return 0;
    prof_mark(EV_QCLUSTER, qs, EV_START);
    joinable = hipEventRecord(aux->join, qs) == hipSuccess;
    return joinable || r ? r : fail(ADACLUSTER_E_INTERNAL, "stream join failed");
  };
  int kc_bound = capacity(p);
  auto keys = [&](const auto& beside) {
    return run_kcluster(p, w, st, K, k_labels, k_centroids, k_assign_centroids, k_bmin, k_bmax, k_sizes, k_count, full_flag,
                        o.k_stage_offs, o.k_stage_of, tau_used, &kc_bound, beside);
  };
  rc = q_first ? queries(true) : 0;
  if (!rc) rc = keys(queries);
  prof_mark(EV_KCLUSTER, st, EV_START);
  if (!joinable) return drained(rc ? rc : ADACLUSTER_E_INTERNAL);
  if (hipStreamWaitEvent(st, aux->join, 0) != hipSuccess) return drained(fail(ADACLUSTER_E_INTERNAL, "stream join failed"));
  if (rc) return rc;                        // (what was queued on the second stream has been joined)
  prof_mark(EV_JOIN, st);
  const float scale = p->softmax_scale > 0.f ? p->softmax_scale : 1.0f / sqrtf((float)p->d);
  int32_t* const sel_keys = plan_reads_lengths(p->q_clusters) ? w.sel_keys : nullptr;
  rc = launch_select(st, p->H, p->q_clusters, capacity(p), p->d, p->score_mode, p->select_mode, p->topk, p->top_p,
                     scale, q_centroids, q_mean_norm, k_centroids, k_bmin, k_bmax, k_sizes, k_count, full_flag,
                     sel_idx, sel_cnt, kc_bound, w.scores, sel_keys);
  if (rc) return drained(rc == ADACLUSTER_E_INTERNAL ? fail(rc, "HIP launch failed: %s", hipGetErrorString(hipGetLastError())) : rc);
  prof_mark(EV_SELECT, st, EV_JOIN);
  // both label sorts were left in the workspace by the clustering steps
  rc = run_plan_attention(p, w, st, Q, O, k_count, sel_idx, sel_cnt, sel_keys, EV_SELECT, K, V);
  return rc ? drained(rc) : 0;
}

int adacluster_dense_attn(const adacluster_params* p, const void* Q, const void* K, const void* V, void* O,
                          void* ws, size_t ws_bytes, void* stream) {
  int rc = check_params(p);
  if (rc) return rc;
  if (!Q || !K || !V || !O) return fail(ADACLUSTER_E_BADARG, "dense_attn: NULL tensor pointer");
  WS w;
  if ((rc = check_ws(p, ws, ws_bytes, &w))) return rc;
  const Dims D = dims_of(p);
  hipStream_t st = (hipStream_t)stream;
  const float scale = p->softmax_scale > 0.f ? p->softmax_scale : 1.0f / sqrtf((float)D.d);
  prof_begin(st);
  const DenseShape shape = attn_dense_shape(p->dtype, D.d, D.H, D.N);
  RET_IF(launch_plan_dense(st, D.H, D.N, D.maxtiles, shape, w.rng_start, w.rng_pre, w.rng_cnt, w.tiles, w.ntiles, w.merge, w.nmerge,
                           key_row_scale(p), w.krow, attn_krow_stride(D.N)));
  prof_mark(EV_PLAN, st);
  RET_IF(launch_attention(st, p->dtype, D.d, D.H, D.N, 1, shape.BM, (D.N + shape.BM - 1) / shape.BM * shape.pieces, D.maxtiles, scale, Q, K, V, O, nullptr, w.tiles,
                          w.ntiles, w.part_o, w.part_ml, shape.pieces > 1 ? w.merge : nullptr, w.nmerge,
                          w.krow, attn_krow_stride(D.N), w.rng_start, w.rng_pre, w.rng_cnt, 1, nullptr, 0, nullptr));
  prof_mark(EV_ATTN, st);
  return 0;
}

int adacluster_stats_fetch(const adacluster_params* p, void* ws, size_t ws_bytes, adacluster_head_stats* host_stats,
                           void* stream) {
  int rc = check_params(p);
  if (rc) return rc;
  if (!host_stats) return fail(ADACLUSTER_E_BADARG, "stats_fetch: host_stats is NULL");
  WS w;
  if ((rc = check_ws(p, ws, ws_bytes, &w))) return rc;
  const Dims D = dims_of(p);
  hipStream_t st = (hipStream_t)stream;
  RET_IF(launch_attn_stats(st, D.H, D.Cq, D.maxr, D.maxtiles, w.kstate, w.tiles, w.ntiles, w.rng_pre, w.rng_cnt, w.stats));
  if (hipMemcpyAsync(host_stats, w.stats, (size_t)D.H * sizeof(adacluster_head_stats), hipMemcpyDeviceToHost, st) != hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess)
    return fail(ADACLUSTER_E_INTERNAL, "stats_fetch: copy to the host failed: %s", hipGetErrorString(hipGetLastError()));
  return 0;
}

int adacluster_mfma_probe(int32_t iters, float* sink, size_t sink_floats, double* flops, void* stream) {
  if (iters < 1 || !sink || !flops) return fail(ADACLUSTER_E_BADARG, "mfma_probe: iters >= 1, sink and flops must be given");
  RET_IF(launch_mfma_probe((hipStream_t)stream, iters, sink, sink_floats, flops));
  return 0;
}

int adacluster_profile_enable(int on) {
  if (on && !g_prof.enabled) {
    for (int i = 0; i < EV_COUNT; ++i)
      if (hipEventCreate(&g_prof.ev[i]) != hipSuccess) return fail(ADACLUSTER_E_INTERNAL, "hipEventCreate failed");
    g_prof.enabled = true;
  } else if (!on && g_prof.enabled) {
    for (int i = 0; i < EV_COUNT; ++i) (void)hipEventDestroy(g_prof.ev[i]);
    g_prof.enabled = false;
  }
  return 0;
}

int adacluster_profile_read(float* ms) {
  if (!ms) return fail(ADACLUSTER_E_BADARG, "ms is NULL");
  if (!g_prof.enabled) return fail(ADACLUSTER_E_UNSUPPORTED, "profiling is not enabled");
  int prev = -1;
  for (int i = 0; i < EV_STAGES; ++i) {
    if (i > 0) ms[i - 1] = -1.f;
    if (!g_prof.recorded[i]) continue;
    if (hipEventSynchronize(g_prof.ev[i]) != hipSuccess) return fail(ADACLUSTER_E_INTERNAL, "event sync failed");
    const int from = g_prof.from[i] >= 0 ? g_prof.from[i] : prev;
    if (from >= 0 && i > 0) {
      if (hipEventSynchronize(g_prof.ev[from]) != hipSuccess) return fail(ADACLUSTER_E_INTERNAL, "event sync failed");
      float t = 0.f;
      if (hipEventElapsedTime(&t, g_prof.ev[from], g_prof.ev[i]) != hipSuccess)
        return fail(ADACLUSTER_E_INTERNAL, "event elapsed failed");
      ms[i - 1] = t;
    }
    prev = i;
  }
  return 0;
}

}  // extern "C"
