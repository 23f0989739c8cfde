// Host-side launchers of the kernels (each enqueues on the given stream and returns 0 or
// ADACLUSTER_E_INTERNAL).
#pragma once
#include "common.h"

namespace adac {

struct SortScratch {
  int32_t* hist;                     // [H][sort_table_ints]: counts of a segment's labels
  int32_t* lab_a; int32_t* val_a;    // [H][sort_scratch_ints] intermediate pass of the one-workgroup sort
  int32_t* lab_b;                    // [H][sort_scratch_ints] its sorted labels
};
size_t sort_table_ints(int N, int m);    // for heads of up to N items and up to m labels
int sort_scratch_ints(int N);

// Stable sort of the first n_h items of every head by label (labels are indexed by position in
// the item list; the items are token ids from `ulist`, or the positions themselves).
//   n_dev / m_dev: per-head item and label counts read on the device (NULL: n_bound / m_bound)
//   active_dev:    per-head flag; heads with 0 are skipped (NULL: all heads)
// Outputs: perm [H][N] token ids ordered by (label, position); offs [H][offs_stride] with
// offs[j] = first sorted position of label j for j = 0..m_h.  With poff, the clusters are also cut into parts of part_rows
// rows for the centroid reduction: poff [H][offs_stride], and pcl [H][P], the cluster of every part, of heads with more
// than 128 labels.  *poff_done says what was left: 1 poff, 2 pcl as well.  A label count above m_bound is taken as m_bound;
// `foreign`: labels outside [0, m) may occur, and their items go to the end of the order, where no offset points.
int launch_sort(hipStream_t st, int H, int N, int n_bound, int m_bound, const int32_t* labels,
                const int32_t* ulist, const int32_t* n_dev, int n_stride, const int32_t* m_dev, int m_stride,
                const int32_t* active_dev, int active_stride, int32_t* perm, int32_t* offs, int offs_stride,
                const SortScratch& sc, int32_t* poff = nullptr, int part_rows = 0, int32_t* pcl = nullptr, int P = 0,
                int* poff_done = nullptr, int foreign = 0);

// n_bound, m_bound: no head has more points or centres.
int launch_assign(hipStream_t s, int dtype, int d, int H, int N, int n_bound, int m_bound, int mode, int m_const, int cap,
                  const KState* st, const int32_t* ulist, const void* X, const void* cent_lp, const float* bias,
                  int32_t* labels, float* dist2,
                  int32_t* keep_lab = nullptr, float* keep_score = nullptr, const int32_t* seed_lab = nullptr,
                  const float* seed_score = nullptr,
                  const float* tau = nullptr, int32_t* keep_cnt = nullptr, int keep_stride = 0, double* dist_sum = nullptr);
// A pass of a stage of Algorithm 1 with at most pass_sum_centres() centres (bf16; fp32: pass_f32_fits()).  An update pass (out)
// leaves the member sums and counts of every pass_points() points; launch_finalize(blk_cnt = out->bcnt, nb_stride = their number, blk_points) turns them
// into centres, or (`wide`, where combine_fits says so) the next pass does, which then takes them as `prev` (another
// table than its `out`).  The last pass (out NULL) leaves what `end` says.  The first pass may open the stage (`open`): it
// then does what launch_stage_open does, from the survivors that the stage before has left.
constexpr int STAGE_SUM_BLOCKS = 128;   // a stage of at most this many blocks of pass_points() may update from their sums
struct StageSums { float* psum; int32_t* bcnt; };     // [H][m_bound * blocks][d] (fp32 stages: doubles), [H][blocks][pass_sum_centres()]
struct PassEnd {
  float* dist2; int32_t* keep_lab; float* keep_score; double* dist_sum;      // the last three as in launch_assign, or NULL
  const float* tau; int32_t* keep_cnt; int keep_stride; int32_t* surv; int32_t* stage_of; int stage;   // survivors of a stage whose threshold is known (keep_cnt, else NULL)
};
struct StageRules { int n_max, m0, m_min, max_stages, u_min; };      // of the loop of Algorithm 1
struct StageFilter; struct StageReport;
struct StageOpening {
  const StageRules* rules; const KState* in; KState* out; const StageFilter* filter /* NULL: the first stage */; const StageReport* report;
  int n_before;                        // no head has more points in the stage that ends
};
int pass_sum_centres();
int pass_points(int dtype, bool wide);
bool pass_f32_fits(int d, int N, int m0);                  // fp32: passes with block sums in all stages of a call, centres formed by the next pass (`wide`) or launch_form_centres
int pass_f32_rows(int d, int N, int m0);                   // most rows of one of their tables in a head of N points
bool combine_fits(int d, int heads, int n_bound, int m_bound);
bool pass_f32_combines(int d, int heads, int n_bound, int m_bound);
bool wide_fills(int heads, int n_bound);      // whether passes without `prev` take `wide` as well
int launch_stage_pass(hipStream_t s, int dtype, int d, int H, int N, int n_bound, int m_bound, int cap, const KState* st, const int32_t* ulist,
                      const void* X, void* cent_lp, float* cent_f32, float* bias, bool wide, const StageSums* prev, const StageSums* out,
                      const PassEnd* end, const StageOpening* open);
int launch_form_centres(hipStream_t s, int d, int H, int n_bound, int m_bound, int cap, const KState* st, const StageSums& sums, void* cent_lp,
                        float* cent_f32, float* bias);
int launch_seg_reduce(hipStream_t s, int dtype, int d, int H, int N, int mode, int m_const, int m_bound, int P,
                      const KState* st, int normalize, int want_box, const void* X, const int32_t* perm,
                      const int32_t* offs, int offs_stride, int32_t* poff, int32_t* pcl, float* psum, float* pnorm, float* pmin,
                      float* pmax, int poff_ready /* what launch_sort left, 1 or 2 */);
int reduce_part_rows();
// What the last launch of a key clustering leaves of its state: the state itself at `home`, and the outputs that are copies
// of it (NULL: not asked for).
struct StateExport {
  KState* home; int32_t* k_count; int32_t* full_flag; int32_t* stage_offs; const float* tau; float* tau_used;
};
int launch_finalize(hipStream_t s, int dtype, int d, int H, int mode, int m_const, int m_bound, int P, int cap,
                    int master_stride, const KState* st, int spherical, int update_assign, int want_box,
                    const int32_t* offs, int offs_stride, const int32_t* poff, const float* psum, const float* pnorm,
                    const float* pmin, const float* pmax, float* master, void* assign_lp, float* assign_f32,
                    float* bias, float* out_cent, const float* fallback, int32_t* out_sizes,
                    float* out_mean_norm, float* out_bmin, float* out_bmax, const int32_t* blk_cnt = nullptr,
                    int nb_stride = 0, int blk_points = 0 /* of a block; 0: nb_stride blocks in every head */, const StateExport* ex = nullptr);
// Label sort (perm, offs as launch_sort leaves them) and final statistics (launch_finalize, update_assign = 0) in one launch:
// cluster_stats_fits() says when.
bool cluster_stats_fits(int dtype, int d, int H, int N, int m_bound, bool keys);
int launch_cluster_stats(hipStream_t s, int dtype, int d, int H, int N, int mode, int m_const, int m_bound, int cap, const KState* st,
                         int spherical, int want_box, const void* X, const int32_t* labels, int32_t* perm, int32_t* offs, int offs_stride,
                         float* out_cent, const float* fallback, int32_t* out_sizes, float* out_mean_norm, float* out_bmin,
                         float* out_bmax, const StateExport* ex);
// Centroid update of a running stage (state mode 1) in one launch, fp32 inputs: every centre's workgroup scans the
// stage's label list (`ulist` NULL: positions are tokens), so it is for few points and centres only:
// direct_update_fits() says when.  Writes what launch_finalize(update_assign = 1) writes.
bool direct_update_fits(int dtype, int n_bound, int m_bound);
int launch_update_direct(hipStream_t s, int d, int H, int N, int m_bound, int cap, int master_stride, const KState* st,
                         const int32_t* labels, const int32_t* ulist, const void* X, float* master, void* assign_lp,
                         float* assign_f32, float* bias);
// One pass of a k-means with at most pass_sum_centres() centres in one read of the points (bf16):
// assignment and (weighted) centroid sums together.  psum [H][m * NP][d], pcnt [H][NP][pass_sum_centres()]
// with NP = qpass_walks(N); launch_finalize(..., blk_cnt = pcnt, nb_stride = NP) turns them into centres.
int qpass_walks(int N);
int launch_qpass(hipStream_t s, int d, int H, int N, int m, int cap, int weighted, const void* X, const void* cent_lp,
                 const float* bias, float* psum, int32_t* pcnt);
// (warm: the states that a warm-started key clustering opens, with k_count and full_flag of the call before; NULL otherwise)
int launch_init_centroids(hipStream_t s, int dtype, int d, int H, int N, int m_const, int m_bound,
                          KState* warm, const int32_t* k_count, const int32_t* full_flag, int spherical, int source_master, int cap,
                          int master_stride, const void* X, float* master, void* assign_lp, float* assign_f32,
                          float* bias);
int launch_tau_abs(hipStream_t s, float tau_abs, float* tau_out);
// What the end of a stage leaves behind for launch_stage_open: squared distances of its last pass and the survivors per
// `items` points (launch_assign with keep_cnt counts per stage_points_per_count(), launch_keep_count per its own).
struct StageFilter {
  const float* dist2; const float* tau; const int32_t* cnt; int cnt_stride; int items;
  const int32_t* uin /* NULL: every token */; int32_t* uout; int32_t* stage_of /* may be NULL */; int stage;
  const int32_t* surv;                 // [H][N] the survivors of every `items` points, from where those start (NULL: not left)
};
struct StageReport { int32_t* sums; int32_t* slot /* mapped host memory, or NULL */; int epoch; };
int stage_points_per_count(int dtype);
// The threshold (with dist_sum, what launch_assign left; NULL: `tau` holds it) and the survivors of the first stage.
int launch_keep_count(hipStream_t s, const KState* st, int H, int N, const float* dist2, const double* dist_sum, int sums, float factor,
                      float* tau, int32_t* cnt, int cnt_stride, int32_t* surv /* NULL: counts alone */, int32_t* stage_of, int* items);      // sums: per head
// Filter of the stage that ends (f; NULL: none, the first stage opens), head of the loop of Algorithm 1, initial centres of
// the stage that opens.  n_bound, m_bound: no head has more points in the stage that ends, or centres in the one that opens.
// The state goes from `in` to `out`, which must differ; report: 4 device integers, and the host's slot, which gets {active heads,
// max |U|, max m_t, epoch}, the epoch behind the rest.
int launch_stage_open(hipStream_t s, int dtype, int d, int H, int N, int cap, const StageRules& rules, int n_bound, int m_bound,
                      const KState* in, KState* out, const StageFilter* f, const StageReport& report, const void* X, void* assign_lp,
                      float* assign_f32, float* bias);
// Every remaining stage of Algorithm 1 in one launch, one workgroup per head (bf16 only).  Valid once every
// active head has at most small_stage_points() unassigned points and small_stage_centres() centres per
// stage, and never for stage 0.  f: the stage before has not been closed; it had at most n_before points a head, and left its
// survivors (sums 0) or, the first stage, distances and what the threshold is formed from: dist_sum, `sums` a head, as in
// launch_keep_count, where small_forms_tau().  NULL: the stage has been opened.
int small_stage_points(int d, int heads);      // heads: still active
int small_stage_centres();
bool small_forms_tau(int H, int sums);
int launch_kstages_small(hipStream_t s, int d, int H, int N, int cap, const StageRules& r, int iters, KState* st, float* tau,
                         int32_t* ulist0, int32_t* ulist1, const void* X, void* cent_lp, float* assign_f32, float* bias,
                         int32_t* stage_of, const StageFilter* f, int n_before, const double* dist_sum, int sums, float factor);
int launch_mse(hipStream_t s, int dtype, int d, int H, int N, int cap, const void* X, const int32_t* labels,
               const float* cent, double* part, float* mse);
int launch_fill_i32(hipStream_t s, int32_t* p, size_t n, int32_t v);

int launch_select(hipStream_t s, int H, int Cq, int cap, int d, int score_mode, int select_mode, int topk,
                  float top_p, float scale, const float* q_cent, const float* q_mean_norm, const float* k_cent,
                  const float* k_bmin, const float* k_bmax, const int32_t* k_sizes, const int32_t* k_count,
                  const int32_t* full_flag, int32_t* sel_idx, int32_t* sel_cnt, int kc_max, double* scores,   // scores: scratch [H][Cq][cap]
                  int32_t* sel_keys /* [H][Cq] keys of the selected clusters and an integer that becomes 0, or NULL */);

int attn_block_rows(int dtype, int d, int N, int Cq);   // queries per workgroup of the attention launch
int attn_block_rows_min(int dtype);
int attn_block_rows_max(int dtype);
int launch_quest_scores(hipStream_t s, int dtype, int form, int clamp, int H, int Lq, int Lk, int d, const void* Q,
                        const void* Rp, const void* Rn, float* S);
// register-only loop of bf16 MFMAs on every SIMD of the chip (measures what the matrix cores sustain)
int launch_mfma_probe(hipStream_t s, int iters, float* sink, size_t sink_floats, double* flops);
int attn_f32_splits(int H, int N, int Cq);   // most pieces a key list of the fp32 kernel may go in
int attn_tile_record();      // ints per query-tile record
int attn_most_tiles(int dtype, int N, int Cq, int BM, int maxtiles);
int attn_split_slots();      // partial slots per head for the chunks of cut key lists (also extra tile records)
bool plan_reads_lengths(int Cq);   // whether launch_plan_sparse has a use for the lengths of the lists
int launch_plan_sparse(hipStream_t s, int dtype, int d, int H, int Cq, int cap, int maxr, int maxtiles, int BM,
                       const int32_t* q_offs, int q_offs_stride, const int32_t* k_offs, int k_offs_stride,
                       const int32_t* k_count, const int32_t* sel_idx, const int32_t* sel_cnt,
                       int32_t* rng_start, int32_t* rng_pre, int32_t* rng_cnt, int32_t* tiles, int32_t* ntiles,
                       int32_t* merge, int32_t* nmerge, int row_scale, int32_t* krow, size_t kstride, const int32_t* perm_k, int N,
                       const int32_t* lengths /* [H][Cq] keys of every list, or NULL: not known beforehand */,
                       int segs /* attn_deal_segs() */, int most /* attn_most_tiles() */, int32_t* deal, int32_t* planned /* an integer; with lengths: 0 */);
// Tiles of a sparse launch dealt to the XCDs by work: segments a head (0: dealt by their number), and the integers of its table.
int attn_deal_segs(int dtype, int d, int H, int N, int Cq, bool top_p);
size_t attn_deal_ints(int dtype, int d, int H, int N, int Cq, int segs, int most);
struct DenseShape { int BM, pieces; };       // queries a workgroup, chunks of the key list
DenseShape attn_dense_shape(int dtype, int d, int H, int N);
int launch_plan_dense(hipStream_t s, int H, int N, int maxtiles, DenseShape shape, int32_t* rng_start, int32_t* rng_pre,
                      int32_t* rng_cnt, int32_t* tiles, int32_t* ntiles, int32_t* merge, int32_t* nmerge, int row_scale, int32_t* krow, size_t kstride);
// entries per (head, query cluster) of the table of key rows (times row_scale) that the attention kernels load by
size_t attn_krow_stride(int N);
bool attn_rows_listed(int dtype, int d, int H, int N, int Cq);    // the planning step writes every key row of a list to a table
int launch_attn_stats(hipStream_t s, int H, int Cq, int maxr, int maxtiles, const KState* st, const int32_t* tiles,
                      const int32_t* ntiles, const int32_t* rng_pre, const int32_t* rng_cnt, adacluster_head_stats* out);
int launch_attention(hipStream_t s, int dtype, int d, int H, int N, int Cq, int BM /* as planned */, int most /* tiles of a head */, int maxtiles, float scale,
                     const void* Q, const void* K, const void* V, void* O, const int32_t* perm_q,
                     const int32_t* tiles, const int32_t* ntiles, float* part_o, float* part_ml,
                     const int32_t* merge /* NULL: no cut lists */, const int32_t* nmerge,
                     const int32_t* krow /* NULL: not attn_rows_listed */, size_t kstride, const int32_t* rng_start,
                     const int32_t* rng_pre, const int32_t* rng_cnt, int maxr, const int32_t* perm_k /* NULL: identity */,
                     int segs /* 0: dealt by their number */, int32_t* deal);

}  // namespace adac
