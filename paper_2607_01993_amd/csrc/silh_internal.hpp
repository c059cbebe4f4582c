// Internal interface between the C ABI (silh_api.cpp) and the kernel files.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace silh {

// Rows per unit of the stable counting sort (one wave per unit): 256 while the
// per-unit histograms (units x k ints) stay small, else 1024.
inline int sort_seg(int64_t n, int k) {
  return (n + 255) / 256 * (int64_t)k <= ((int64_t)1 << 26) ? 256 : 1024;
}
// Elements per block of the int32 exclusive scan (256 threads x 8).
constexpr int kScanTile = 2048;
// Members per work item of the W(e_bar) partial sums.
constexpr int kWChunk = 256;   // one member per thread of a 256-thread block
constexpr int kWChunkWide = 256;  // d > 128: one member per thread as well
// Sample rows of each cluster are padded to a multiple of this.
constexpr int kSamplePad = 32;
// Rows per Phase-2 block in the VALU kernel.
constexpr int kP2Rows = 256;

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ---- cluster index -------------------------------------------------------
// per-unit label histograms uh [k][units] (label-major); *bad = 1 if a label
// is outside [0, k) (bad may be null: such a label is counted nowhere)
void launch_unit_hist(hipStream_t st, const int32_t* labels, int n, int k, int seg, int32_t* uh,
                      int32_t* perm = nullptr, int32_t* slab = nullptr);
// uh[u][j] <- label j's rows before unit u; counts[j] = |C_j|
void launch_unit_scan(hipStream_t st, int32_t* uh, int units, int k, int32_t* counts);
// stable scatter: rows of label j go to off[j] + uh[u][j] + (rank inside the unit)
void launch_scatter(hipStream_t st, const int32_t* labels, int n, int k, int seg, const int32_t* ubase,
                    const int32_t* off, int32_t* perm, int32_t* slab);
// out[0..n] = exclusive prefix sums of in[0..n), out[n] = total.  tmp holds
// scan_words(n) ints; with `sums` it holds the sums of every 256 values on
// entry (bsum of the kernels below).
inline int64_t scan_words(int64_t n) { return (n + 255) / 256 + 2; }
void launch_scan(hipStream_t st, const int32_t* in, int n, int32_t* out, int32_t* tmp, bool sums = false);
// out[j] = scan[off[j]] for j in [0, k]
void launch_gather_at(hipStream_t st, const int32_t* scan, const int32_t* off, int k, int32_t* out);

// ---- Phase 1 -----------------------------------------------------------------
void launch_f0_flag(hipStream_t st, const int32_t* perm, const int32_t* slab, int n,
                    const int32_t* csize, const double* q, int64_t t, uint64_t seed, int32_t* flag,
                    int32_t* bsum);
// The W pass's work items as launch_f0_items sized them (cap 0: none).
struct W0Items {
  const int32_t *off = nullptr, *f0_off = nullptr, *citem_first = nullptr;
  const int64_t* ibase = nullptr;
  const int32_t* meta = nullptr;
  int32_t* items = nullptr;
  int k = 0, chunk = 0, cap = 0;
};
// rows past `cap` (the capacity of f0_gid / f0_cl / f0X / f0N) are not written;
// f0N (cosine, else null): the rows' norms; A: also the W pass's work items
// (A.cap slots, the unused ones empty)
void launch_f0_pack(hipStream_t st, const int32_t* perm, const int32_t* slab, const int32_t* flag,
                    const int32_t* pos, int n, const float* X, int d, int DM, int cap, int64_t* f0_gid,
                    int32_t* f0_cl, double* f0X, double* f0N = nullptr, const W0Items& A = {});
// float64 distances from the members of each cluster to its initial-sample
// rows, kept by the W pass for the draw (which then reads them instead of
// evaluating them again): the distance of the member at sorted position i of
// cluster j to F0_j's e-th row is at d[base[j] + e |C_j| + (i - off[j])].
// With d null, or *use == 0 (set on the device when the distances did not fit
// their capacity), nothing is kept and the draw evaluates the distances.
struct DistStore {
  double* d = nullptr;
  const int64_t* base = nullptr;  // [k]
  const int32_t* off = nullptr;   // [k + 1] cluster offsets
  const int32_t* use = nullptr;   // device flag
};
// one block per work item: item = (cluster, first sorted pos, end sorted pos,
// first F0 index of the cluster, |F0_j|, base in `partial`)
// f0X rows have stride DM (zero-padded)
void launch_w_partial(hipStream_t st, int metric, int DM, const int32_t* items, int nitems,
                      const int32_t* perm, const float* X, int d, const double* f0X, const double* f0N,
                      double* partial, DistStore ds = {});
// F0 blocks at most; those at or past f0_off[k] return at once
void launch_w_final(hipStream_t st, const int32_t* f0_cl, int F0, const int32_t* f0_off, int k,
                    const int32_t* citem_first, const int32_t* citem_count, const int32_t* items,
                    const double* partial, double* W);
void launch_draw(hipStream_t st, int metric, int DM, int sampler, const int32_t* perm,
                 const int32_t* slab, int n, const float* X, int d, const int32_t* csize, int64_t t,
                 uint64_t seed, const int32_t* f0_off, const double* f0X, const double* W,
                 double* p_gid, int32_t* flag, DistStore ds = {}, int32_t* bsum = nullptr);
void launch_fill_all(hipStream_t st, const int32_t* perm, int n, double* p_gid, int32_t* flag,
                     int32_t* bsum = nullptr);
// rn[i] = 1 / |X_i| in float32 (fused chain in coordinate order, correctly
// rounded square root and division), 0 for a zero row
void launch_rnorm(hipStream_t st, const float* X, int n, int d, float* rn);
// the launch_pack mode of a metric (metric ids as in silh_metric: 1 cosine,
// 3 Canberra)
inline int pack_mode(int metric) { return metric == 1 ? 1 : (metric == 3 ? 2 : 0); }
// Scatter the selected elements into the cluster-blocked, padded sample.
// mode 0: raw coordinates; 1: rows times rn (unit L2 norm, cosine; weight and
// coordinates 0 for a row that is not finite); 2: raw
// coordinates with aux32 = 1 for a row holding a coordinate of magnitude
// above 2^62 (or not finite), else 0 (Canberra; see k_phase2_valu.hip).  Rows at
// or past `cap` (the capacity of the packed arrays) are not written.  Every
// other row in [0, sp_off[k]) is written, the padding rows of each cluster
// block as id -1 with zero weight, aux and coordinates: no prior clear.
void launch_pack(hipStream_t st, const int32_t* perm, const int32_t* slab, const int32_t* flag,
                 const int32_t* pos, int n, int k, const float* X, int d, int DM, const double* p_gid,
                 const int32_t* s_off, const int32_t* sp_off, int mode, const float* rn, int cap,
                 int64_t* gid_view, int32_t* gid_pk, float* w32, float* aux32, float* Y32);

// ---- Phase 2 -----------------------------------------------------------------
struct P2Args {
  const float* X;
  int n, d;
  const int32_t* labels;
  const float* Y;      // [S_pad][DM]
  const float* w;      // [S_pad]
  const float* aux;    // [S_pad] Canberra: the row's form flag (launch_pack)
  const int32_t* sp_off;  // [k+1] padded sample offsets
  const int32_t* cnt;     // [k] |F_j|
  const int32_t* csize;   // [k] |C_j|
  int k;
  float* a;
  float* b;
  float* s;
  float* What;          // [n][k] or null
  double* bpart;        // [ceil(n / rows per partial)]
  double* Wpart = nullptr;  // [n][k] float64, for the split vector-ALU pass (d > 128)
  const float* rn = nullptr;  // [n] cosine: reciprocal row norms (launch_rnorm) of X's rows
  const unsigned char* cstat = nullptr;  // cosine: the clusters' records (launch_cos_stats)
  const float* cself = nullptr;    // cosine, fp8: launch_cos_self's values by element id
  const int32_t* egid = nullptr;   // element ids of the rows of X (null: row i is element i)
  // matrix-core path and tables: the order in which the rows are taken (a
  // permutation of [0, n), null: as they lie); matrix-core path: the clusters each group of 32 of them
  // needs (launch_bounds; null: every cluster)
  const int32_t* perm = nullptr;
  const uint32_t* mask = nullptr;
  // matrix-core path: split blocks (mfma_split), whose bpart holds a partial per
  // 32 elements, for launch_mean's quads
  bool split = false;
};
// One request's Phase-2 launch as a work source of a multi-request launch
// (the arguments of P2Args and of the matrix-core operands, in device memory).
struct P2Job {
  const float* X;
  const int32_t* labels;
  const void* Ym;        // matrix-core operands (null on the vector-ALU path)
  const float* w;
  const int32_t* sp_off;
  const int32_t* cnt;
  const int32_t* csize;
  const float* mu;
  float* a;
  float* b;
  float* s;
  float* What;
  double* bpart;
  const float* Y32;
  const float* aux;
  const int32_t* perm;
  const uint32_t* mask;
  int n, d, k, pad0;
};
// returns false if (metric, d) has no VALU kernel
bool launch_phase2_valu(hipStream_t st, int metric, int DM, const P2Args& a);
// Multi-request launches: workgroup i runs work item items[i] = (index into
// jobs, block of that job's own launch).  The vector-ALU form covers the
// one-pass shapes with the row in registers (phase2_valu_jobs_ok); blocks
// are phase2_valu_rows / phase2_mfma_rows * pb elements.
bool launch_phase2_valu_jobs(hipStream_t st, int metric, int DM, const P2Job* jobs, const int2* items, int nitems);
bool phase2_valu_jobs_ok(int metric, int DM);
bool launch_phase2_mfma_jobs(hipStream_t st, int prec, int DM, int shape, const P2Job* jobs, const int2* items,
                             int nitems);
int phase2_valu_dm(int d);   // padded dimension used by the VALU kernel, 0 if unsupported
// elements per block (and per partial of the mean) of the VALU kernel
int phase2_valu_rows(int metric, int DM);
// d > 128 Manhattan / Canberra run as two coordinate halves and need
// P2Args::Wpart ([n][k] float64 scratch)
bool phase2_valu_split(int metric, int DM);

// MFMA path (Euclidean).  prec: 0 float32, 1 bf16 operands.
int mfma_kp(int prec, int DM);   // contraction length of a packed row
int mfma_row_bytes(int prec, int DM);  // bytes per packed row (operands, LDS-path tail)
// mu: [k][KP] centres, zero beyond DM, then [k] squared radii of the
// clusters' packed samples (the largest |y~_q|^2), mfma_mu_floats
// floats in all
size_t mfma_mu_floats(int prec, int DM, int k);
// With rec non-null also the bound records (below).
void launch_center(hipStream_t st, int prec, int DM, const float* Y32, const float* w, const int32_t* sp_off,
                   const int32_t* cnt, const int32_t* csize, int k, float* mu, float* rec);
// packs rows [0, min(S_pad, sp_off[k])) (w: weights of the packed rows,
// copied into the rows' tails on the LDS path)
// With A: also the bounds' probe over A's elements and records.
struct ProbeArgs {
  const float* X = nullptr;
  const int32_t *labels = nullptr, *perm = nullptr;
  float* rec = nullptr;  // null: no probe
  int n = 0, d = 0;
};
bool launch_pack_mfma(hipStream_t st, int prec, int DM, const float* Y32, const float* w, const int32_t* sp_off,
                      const int32_t* cnt, int k, float* mu, int S_pad, void* Ym, const ProbeArgs& A = {});
// elements per float64 partial of the sum of s_hat written by the MFMA
// Phase-2 kernel (independent of its block shape)
int phase2_mfma_rows(int prec, int DM);
// Block shapes (ids): 1 one 32-element block per wave, 2 two blocks per wave
// (d <= 64), 3 one block with the other number of tiles per LDS
// stage (the LDS-staged shapes only).  The default choice of blocks per wave:
int mfma_pb_default(int prec, int DM);
int mfma_pb_max(int prec, int DM);
// whether a launch over n elements splits the clusters over a block's waves
bool mfma_split(int prec, int DM, int64_t n, int k);
bool mfma_lds_path(int prec, int DM);
// the packed rows hold three bf16 pieces of each float32 coordinate
bool mfma_three_pieces(int prec, int DM);
// the shape ids valid for (prec, DM) into ids[0..2]; returns their count
int mfma_shapes(int prec, int DM, int* ids);
bool launch_phase2_mfma(hipStream_t st, int prec, int DM, const P2Args& A, const float* mu, const void* Ym,
                        int shape);

// Bounds on the Euclidean sums (k_phase2_bounds.hip): a record per cluster
// (bound_rec_floats floats in all, by launch_center), then for every
// group of 32 elements (in perm order, null: as they lie) a mask of the
// clusters its scores need, bit j of word [group][j / 32]
// the probe (kBoundProbe blocks of 64 elements, by launch_pack_mfma) leaves the
// number of clusters that each of its blocks needs behind the records
constexpr int kBoundProbe = 32;
size_t bound_rec_floats(int DM, int k);
// (a head of kBoundHead words before them: head[kBoundFlag] = 1 if the masks are
// not to be used)
constexpr int kBoundHead = 64, kBoundFlag = 0;
size_t bound_mask_words(int64_t n, int k);
// buf: bound_mask_words words.  Returns the masks in it.
const uint32_t* launch_bounds(hipStream_t st, int DM, const float* X, int n, int d, const int32_t* labels,
                              const int32_t* perm, const float* rec, int k, int limit, uint32_t* buf);
// How scores of n elements against a sample of about S = min(n, k t) rows go
// through the bounds: not at all, or with a probe first: whether the clusters it finds
// needed, of every 128 groups' (limit), leave the rest worth the bounds' cost
struct BoundPlan {
  bool use = false;
  int limit = -1;  // -1: no probe
};
BoundPlan bound_plan(int prec, int DM, int64_t n, int k, int64_t S);

// Cosine (every operand type; prec as above, float32 arithmetic for the
// vector-ALU precision too): the clusters' samples collapsed into one record
// each (k records of cos_stat_bytes), then one pass over the elements.
constexpr int kCosRows = 64;  // elements per block (and per partial of the mean)
size_t cos_stat_bytes(int DM);
void launch_cos_stats(hipStream_t st, int prec, int DM, const float* Y32, const float* w, const float* aux,
                      const int32_t* sp_off, const int32_t* cnt, int k, unsigned char* stat);
// fp8 only: self [n] (zeros, then the sampled elements' values); rows at or
// past `cap` of the packed sample are not read
void launch_cos_self(hipStream_t st, int DM, const float* Y32, const float* w, const int32_t* gid_pk,
                     const int32_t* sp_off, int k, int cap, const unsigned char* stat, int n, float* self);
// pieces: the elements in pieces of about a millisecond with a wait between them
// (tab_plan)
bool launch_phase2_cos(hipStream_t st, int prec, int DM, const P2Args& A, bool pieces = false);

// Manhattan and Canberra by per-coordinate tables (k_phase2_tab.hip): whether
// they pay for n elements against clusters of about min(t, n / k) sample rows
bool tab_pays(int metric, int64_t n, int k, int64_t t);
constexpr int kTabScore = kP2Rows;  // elements per partial of the mean (as the direct kernel)
struct TabPlan {
  int64_t chunks = 0, group = 0, rows = 0;  // tables' chunks (at most), chunks and elements taken at once
  size_t knots = 0;                         // knots of a group's tables (all coordinates)
  int rw = 0, max_knots = 0;                // floats per record, knots of the longest table
  bool wait = false;                        // wait for the stream between the pieces
};
struct TabBufs {
  int32_t* chunk = nullptr;   // [4 chunks]
  int32_t* cfirst = nullptr;  // [k + 1]
  unsigned char* head = nullptr;  // [group d tab_head_bytes]
  float* Y = nullptr;         // [knots]
  double* G = nullptr;        // [2 knots]
  float* C = nullptr;         // [2 knots], Canberra
  uint16_t* L = nullptr;      // [group d tab_cells]
  float* XT = nullptr;        // [rows d]
  double* Wd = nullptr;       // [k rows]
};
// S_pad, max_rows: packed sample rows and the largest cluster's (or bounds);
// pieces: the elements in pieces of about a millisecond with a wait between
// them (streams outnumber the hardware queues, so that another stream's short
// kernels may sit behind a long launch; the results are the same)
TabPlan tab_plan(int metric, int64_t n, int d, int k, int64_t S_pad, int64_t max_rows, bool pieces = false);
size_t tab_head_bytes();
size_t tab_cells();
size_t tab_bytes(const TabPlan& p, int k, int d);
bool launch_phase2_tab(hipStream_t st, int metric, int DM, const P2Args& A, const TabPlan& p, const TabBufs& B);

// ---- Phase-2 path of a request ------------------------------------------------
// cosine: the collapsed sums; Euclidean with matrix-core operands: the MFMA
// kernel (float32 operands of d > 128 do not fit its registers); else the
// vector ALUs
enum P2Path { kPathValu = 0, kPathMfma = 1, kPathCos = 2 };
int phase2_path(int metric, int prec, int DM);
// operand type of the matrix-core and cosine kernels: 0 float32, 1 bf16, 2 fp8
int operand_type(int prec);
int phase2_rows(int path, int metric, int mprec, int DM);

// ---- global mean -------------------------------------------------------------
// quads: bpart holds nq partials, of which every four are added first (in order)
// (with status, the clustering's status word goes to *status_out)
void launch_mean(hipStream_t st, const double* bpart, int nb, int64_t n, double* out, int nq = 0,
                 const int* status = nullptr, int32_t* status_out = nullptr);

// ---- device-side sizes for the capturable pipeline (k_graph.hip) ------------
// bits of a clustering's status word
constexpr int kStatusLabel = 1;    // a label outside [0, k) (set by k_index_sizes)
constexpr int kStatusEmpty = 2;    // fewer than two nonempty clusters
constexpr int kStatusF0 = 4;       // F0 larger than its capacity
constexpr int kStatusPartial = 8;  // W(e_bar) partial sums larger than their capacity
constexpr int kStatusSample = 16;  // padded sample larger than its capacity
void launch_fill_i32(hipStream_t st, int32_t* p, int64_t count, int32_t v);
// off[0..k] = exclusive prefix sums of csize; q[j] = min(1, (2/|C_j|) lnterm)
void launch_index_sizes(hipStream_t st, const int32_t* csize, int n, int k, double lnterm, int32_t* off, double* q,
                        int* status);
// f0_off[j] = pos[off[j]], clamped to f0_cap, and the W work items' sizes:
// per-cluster first item / count and partial bases;
// with dbase non-null also the bases of the kept distances (DistStore) and
// meta[1] = 1 when they fit dist_cap doubles.  The capacity bits go into
// *status: ORed in, or with assign_status the word is set to them (a status
// word of its own, which then needs no clear before the launch)
void launch_f0_items(hipStream_t st, const int32_t* csize, const int32_t* off, const int32_t* pos, int32_t* f0_off,
                     int k, int64_t t, int chunk, int f0_cap, int64_t part_cap, int32_t* citem_first,
                     int32_t* citem_count, int64_t* ibase, int32_t* meta, int* status, int64_t* dbase = nullptr,
                     int64_t dist_cap = 0, bool assign_status = false);
// capacity (doubles) of the kept distances for n elements, k clusters and
// ln(5k/delta): about 1.25 times their expected count, at most 2^27
int64_t dist_capacity(int64_t n, double lnterm);
// s_off[j] = pos[off[j]], cnt[j] = |F_j|, sp_off = offsets of the blocks padded to kSamplePad rows
void launch_sample_sizes(hipStream_t st, const int32_t* pos, const int32_t* off, int32_t* s_off, int k, int s_cap,
                         int32_t* cnt, int32_t* sp_off, int* status);
void launch_put_status(hipStream_t st, const int* status, int32_t* out);

// ---- host-side helpers shared by the C-ABI files ----------------------------
}  // namespace silh
#include "../../include/silh.h"
namespace silh {
// the argument checks of silh_sample_init; *t receives the sample size used
silh_status validate_params(const silh_params* prm, const float* X, const int32_t* labels, int64_t* t);
// the argument checks of silh_exact (t, eps, delta, sampler and seed unused)
silh_status validate_exact_params(const silh_params* prm, const float* X, const int32_t* labels);
// padded row width of the packed sample for dimension d (0 if unsupported)
int dm_for(int d);
// sets the thread's silh_last_error message and returns st
silh_status set_error(silh_status st, const char* msg);

// ---- one request's Phase 2 inside a multi-request launch (serving) ---------
// The kernel class of a request's Phase 2 (requests of one class share a
// launch) and its work: `blocks` work items of `rows` elements, each against
// the S_pad packed sample rows.
struct P2Class {
  int mfma, metric, prec, DM, pb, rows;  // prec: 0 float32, 1 bf16, 2 fp8 operands, -1 vector ALU; pb: shape id
  int64_t blocks, S_pad;
};
// After a successful silh_pps_sample: ctx's Phase 2 (no per-element outputs;
// the block partials of the mean stay in the context) as a job of the
// multi-request launch.  False when its shape has no multi-request kernel
// (vector ALU with d > 128): then silh_scores runs it alone.
bool phase2_job(silh_ctx* c, P2Job* job, P2Class* cls);
// the autotuner's shape for ctx's Phase 2 (timing the shapes on ctx's data
// when its key is new; the built-in shape on the vector ALUs or in mode 0);
// split: in split blocks where the launch takes them (mfma_split)
int tuned_shape(silh_ctx* c, bool split);
// padded sample rows of a sampled context (the tuner's size key), else 0
int64_t sample_rows(const silh_ctx* c);
// launch work items of requests of one class (workgroup i runs items[i])
bool launch_phase2_class(hipStream_t st, const P2Class& cls, const P2Job* jobs, const int2* items, int nitems);
// whether ctx's later Phase-2 launches leave room for other streams' work
void set_pieces(silh_ctx* c, bool on);
// whether ctx goes without the buffers that only save work: tables, bounds,
// operand rows of three pieces (set before silh_pps_sample)
void set_lean(silh_ctx* c, bool on);
// after the job's items have all run: the Eq. 9 mean from its block partials
// (on the context's stream; synchronises it)
silh_status phase2_job_mean(silh_ctx* c, double* mean);

// ---- cohesion / separation numerators from W_hat [n][k] ---------------------
constexpr int kCohSepMaxBlocks = 1024;
int coh_sep_blocks(int n);
// cpart/spart[block] = float64 partial sums of W_hat[e][own(e)] and of
// W_hat[e][j] over j > own(e)
void launch_coh_sep(hipStream_t st, const float* W, int n, int k, const int32_t* labels, double* cpart,
                    double* spart);

// ---- subsampled global estimators (row subsets) ------------------------------
// rows[i] = floor(B_i * n / 2^53), B_i the 53 Philox bits of counter i in the
// row stream
void launch_rows_draw(hipStream_t st, uint64_t seed, int64_t n, int64_t m, int32_t* rows);
// mark[rows[i]] = 1 for every valid entry; *bad = 1 if any entry lies outside [0, n)
void launch_rows_mark(hipStream_t st, const int32_t* rows, int64_t m, int n, int32_t* mark, int* bad);
// flag[i] = mark[perm[i]]: the marked elements in cluster order
void launch_rows_flag(hipStream_t st, const int32_t* mark, const int32_t* perm, int n, int32_t* flag);
// urows[pos[i]] = perm[i] for every flagged i (distinct, in cluster order) and
// slot[perm[i]] = pos[i]
void launch_rows_compact(hipStream_t st, const int32_t* flag, const int32_t* pos, const int32_t* perm, int n,
                         int32_t* urows, int32_t* slot);
// Xs[i] = X[urows[i]], ls[i] = labels[urows[i]]
void launch_rows_gather(hipStream_t st, const float* X, const int32_t* labels, int d,
                        const int32_t* urows, int mu, float* Xs, int32_t* ls);
// a/b/s[i] = a/b/s_u[slot[rows[i]]]; bpart[block] = float64 sum
// of the block's s (blocks of kRowsBlock entries)
constexpr int kRowsBlock = 256;
void launch_rows_expand(hipStream_t st, const int32_t* rows, int64_t m, const int32_t* slot, const float* au, const float* bu, const float* su, float* a, float* b, float* s,
                        double* bpart);

// ---- diagnostics -------------------------------------------------------------
void launch_uniform(hipStream_t st, uint64_t seed, int64_t gid0, int64_t count, uint32_t stream_id,
                    double* out);

}  // namespace silh
