// silh_exact_noalloc: the exact silhouette of silh_exact with every scratch
// buffer carved out of one static device array, for callers that cannot
// allocate device memory.
//
// The work is the pipeline of silh_exact (cluster index, F_j = C_j with
// p = 1, packing, Phase 2, the mean) with every size computed on the device
// (the kernels of the captured-graph path), so nothing is read back before
// the end and nothing is allocated: the library's own buffers are slices of
// `scratch`, a file-scope device array of kScratchBytes.  Each device holds
// its own copy of the array, at its own address, from the first call on it
// until the process ends; host code reaches it only through the address
// hipGetSymbolAddress returns for the current device (the array's name is a
// host-side stand-in, not a device address).  The array keeps the previous
// call's contents: every slice that must start at a known value is filled by
// a kernel here (no memset, so the sequence is also valid inside a captured
// stream).  Calls on one device share the array: the library serialises the
// calls of one process per device (a lock held until the call has
// synchronised its stream), and calls that overlapped on one device (from
// work the caller enqueued around them on other streams reading the same
// slices) would race.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <mutex>

#include "silh_internal.hpp"

using namespace silh;

namespace {

constexpr size_t kScratchBytes = (size_t)256 << 20;  // 256 MiB per device
constexpr int kMaxDevices = 64;

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

// the cosine path's cluster records, at their largest (k = 4096, d = 256);
// an array of their own, so that they take nothing from the capacity above
constexpr size_t kRecordBytes = (size_t)4096 * (64 + 256 * 12);
static __device__ __align__(256) unsigned char records[kRecordBytes];

// Rows of three bf16 pieces and their centres (float32 Euclidean, d from 9 to
// 64) are larger than the float32 rows that the capacity counts: they have an
// array of their own, enough for every request that fits the capacity (the
// largest share is d > 32: 432 bytes a row where `scratch` holds at least 564).
constexpr size_t kOperandBytes = (size_t)208 << 20;
static __device__ __align__(256) unsigned char operands[kOperandBytes];

size_t f32_row_bytes(int DM) { return (size_t)(DM + 4) * 4 + (DM > 32 ? 16 : 0); }

std::mutex g_mu[kMaxDevices];
void* g_ptr[kMaxDevices] = {};
void* g_rec[kMaxDevices] = {};
void* g_ops[kMaxDevices] = {};

// The device address of this device's copy of `scratch`, looked up once per
// device (with that device current) and kept.
silh_status scratch_for(int dev, unsigned char** out, unsigned char** rec, unsigned char** ops) {
  if (!g_ptr[dev]) {
    void *p = nullptr, *r = nullptr, *o = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr ||
        hipGetSymbolAddress(&r, HIP_SYMBOL(records)) != hipSuccess || r == nullptr ||
        hipGetSymbolAddress(&o, HIP_SYMBOL(operands)) != hipSuccess || o == nullptr) {
      (void)hipGetLastError();
      return set_error(SILH_E_HIP, "hipGetSymbolAddress of the static scratch array failed");
    }
    g_ptr[dev] = p;
    g_rec[dev] = r;
    g_ops[dev] = o;
  }
  *out = (unsigned char*)g_ptr[dev];
  *rec = (unsigned char*)g_rec[dev];
  *ops = (unsigned char*)g_ops[dev];
  return SILH_OK;
}

// Slices of the scratch array, each 256-byte aligned.  With base == nullptr
// only the total is counted.
struct Slices {
  unsigned char* base = nullptr;
  size_t used = 0;
  template <class T>
  Slices& add(T** p, int64_t count) {
    const size_t bytes = ((size_t)(count > 0 ? count : 1) * sizeof(T) + 255) & ~(size_t)255;
    if (base) *p = (T*)(base + used);
    used += bytes;
    return *this;
  }
};

struct Bufs {
  int *status = nullptr;
  int32_t *uh = nullptr, *csize = nullptr, *off = nullptr, *perm = nullptr, *slab = nullptr;
  double* q = nullptr;
  int32_t *flag = nullptr, *pos = nullptr, *scan_tmp = nullptr, *s_off = nullptr, *sp_off = nullptr,
          *cnt = nullptr;
  double* p_gid = nullptr;
  int64_t* gid_view = nullptr;
  int32_t* gid_pk = nullptr;
  float *w32 = nullptr, *aux32 = nullptr, *Y32 = nullptr, *mu = nullptr;
  unsigned char* Ym = nullptr;
  double *bpart = nullptr, *Wpart = nullptr, *mean = nullptr;
  float* rn = nullptr;
  unsigned char* cstat = nullptr;
  float* cself = nullptr;
  float* brec = nullptr;
  uint32_t* bmask = nullptr;
};

struct Shape {
  int n, d, k, DM, mprec, p2_rows, seg, units;
  bool mfma, split, cos, bounds, split32, pieces;
  int64_t S_cap;
};

void layout(const Shape& s, Slices& sl, Bufs& b) {
  const int64_t n = s.n, k = s.k;
  sl.add(&b.status, 1).add(&b.mean, 1).add(&b.uh, (int64_t)s.units * k).add(&b.csize, k).add(&b.off, k + 1);
  sl.add(&b.perm, n).add(&b.slab, n).add(&b.q, k).add(&b.flag, n).add(&b.pos, n + 1);
  sl.add(&b.scan_tmp, ceil_div(n, kScanTile) + 1).add(&b.s_off, k + 1).add(&b.sp_off, k + 1).add(&b.cnt, k);
  sl.add(&b.p_gid, n).add(&b.gid_view, s.S_cap).add(&b.gid_pk, s.S_cap).add(&b.w32, s.S_cap);
  sl.add(&b.aux32, s.S_cap).add(&b.Y32, s.S_cap * s.DM).add(&b.bpart, ceil_div(n, s.split32 ? 32 : s.p2_rows));
  if (s.mfma) {
    if (s.pieces)
      sl.add(&b.mu, k * (int64_t)(s.DM + 4) + k).add(&b.Ym, s.S_cap * (int64_t)f32_row_bytes(s.DM));
    else
      sl.add(&b.mu, mfma_mu_floats(s.mprec, s.DM, k)).add(&b.Ym, s.S_cap * (size_t)mfma_row_bytes(s.mprec, s.DM));
  }
  if (s.split) sl.add(&b.Wpart, n * k);
  if (s.bounds) sl.add(&b.brec, (int64_t)bound_rec_floats(s.DM, s.k)).add(&b.bmask, (int64_t)bound_mask_words(n, s.k));
  if (s.cos) sl.add(&b.rn, n);
}

}  // namespace

extern "C" silh_status silh_exact_noalloc(const silh_params* prm, const float* X, const int32_t* labels,
                                          silh_stream stream, float* a, float* b, float* s,
                                          double* s_mean_host) {
  {
    const silh_status v = validate_exact_params(prm, X, labels);
    if (v != SILH_OK) return v;
  }
  Shape sh;
  sh.n = (int)prm->n;
  sh.d = prm->d;
  sh.k = prm->k;
  sh.DM = dm_for(prm->d);
  const int path = phase2_path(prm->metric, prm->prec, sh.DM);
  sh.mfma = path == kPathMfma;
  sh.mprec = operand_type(prm->prec);
  sh.p2_rows = phase2_rows(path, prm->metric, sh.mprec, sh.DM);
  sh.pieces = sh.mfma && mfma_three_pieces(sh.mprec, sh.DM);
  sh.split = !sh.mfma && phase2_valu_split(prm->metric, sh.DM);
  sh.cos = path == kPathCos;
  sh.seg = sort_seg(sh.n, sh.k);
  sh.units = (int)ceil_div(sh.n, sh.seg);
  sh.S_cap = (int64_t)sh.n + (int64_t)kSamplePad * sh.k;  // every element, each cluster padded
  sh.split32 = sh.mfma && mfma_split(sh.mprec, sh.DM, sh.n, sh.k);
  // the bounds (the same results) where their buffers fit too
  const BoundPlan plan = sh.mfma ? bound_plan(sh.mprec, sh.DM, sh.n, sh.k, sh.n) : BoundPlan{};
  sh.bounds = plan.use;
  if (sh.bounds) {
    Slices count;
    Bufs dummy;
    layout(sh, count, dummy);
    sh.bounds = count.used <= kScratchBytes;
  }
  {
    Slices count;
    Bufs dummy;
    layout(sh, count, dummy);
    if (count.used > kScratchBytes) {
      char msg[200];
      std::snprintf(msg, sizeof msg,
                    "n=%d, d=%d, k=%d needs %zu bytes of scratch; the static array holds %zu", sh.n, sh.d, sh.k,
                    count.used, kScratchBytes);
      return set_error(SILH_E_ARG, msg);
    }
  }
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    (void)hipGetLastError();
    return set_error(SILH_E_HIP, "no current HIP device");
  }
  std::lock_guard<std::mutex> lk(g_mu[dev]);
  unsigned char *base = nullptr, *rec = nullptr, *ops = nullptr;
  {
    const silh_status v = scratch_for(dev, &base, &rec, &ops);
    if (v != SILH_OK) return v;
  }
  Slices sl;
  sl.base = base;
  Bufs B;
  layout(sh, sl, B);
  if (sh.cos) B.cstat = rec;
  if (sh.cos && sh.mprec == 2) B.cself = (float*)B.pos;  // (read last by the packing)
  if (sh.cos && (size_t)sh.k * cos_stat_bytes(sh.DM) > kRecordBytes)
    return set_error(SILH_E_ARG, "too many clusters for the static record array");
  if (sh.pieces) {
    const size_t rows = ((size_t)sh.S_cap * mfma_row_bytes(sh.mprec, sh.DM) + 255) & ~(size_t)255;
    if (rows + mfma_mu_floats(sh.mprec, sh.DM, sh.k) * sizeof(float) > kOperandBytes)
      return set_error(SILH_E_ARG, "too many rows for the static operand array");
    B.Ym = ops;
    B.mu = (float*)(ops + rows);
  }

  const hipStream_t st = (hipStream_t)stream;
  const int n = sh.n, k = sh.k, d = sh.d, DM = sh.DM;
  const int metric = prm->metric;
  // cluster index; the log term of q is unused here
  launch_unit_hist(st, labels, n, k, sh.seg, B.uh, B.perm, B.slab);
  launch_unit_scan(st, B.uh, sh.units, k, B.csize);
  launch_index_sizes(st, B.csize, n, k, 0.0, B.off, B.q, B.status);
  launch_scatter(st, labels, n, k, sh.seg, B.uh, B.off, B.perm, B.slab);
  if (B.rn) launch_rnorm(st, X, n, d, B.rn);
  // every element sampled with p = 1 (Section 2: the exact sums)
  launch_fill_all(st, B.perm, n, B.p_gid, B.flag);
  launch_scan(st, B.flag, n, B.pos, B.scan_tmp);
  launch_sample_sizes(st, B.pos, B.off, B.s_off, k, (int)sh.S_cap, B.cnt, B.sp_off, B.status);
  launch_pack(st, B.perm, B.slab, B.flag, B.pos, n, k, X, d, DM, B.p_gid, B.s_off, B.sp_off, pack_mode(metric),
              B.rn, (int)sh.S_cap, B.gid_view, B.gid_pk, B.w32, B.aux32, B.Y32);
  P2Args A;
  A.X = X;
  A.n = n;
  A.d = d;
  A.labels = labels;
  A.Y = B.Y32;
  A.w = B.w32;
  A.aux = B.aux32;
  A.sp_off = B.sp_off;
  A.cnt = B.cnt;
  A.csize = B.csize;
  A.k = k;
  A.a = a;
  A.b = b;
  A.s = s;
  A.What = nullptr;
  A.bpart = B.bpart;
  A.Wpart = B.Wpart;
  A.rn = B.rn;
  A.cstat = B.cstat;
  A.cself = B.cself;
  bool ok = true;
  if (sh.cos) {
    launch_cos_stats(st, sh.mprec, DM, B.Y32, B.w32, B.aux32, B.sp_off, B.cnt, k, B.cstat);
    if (B.cself) launch_cos_self(st, DM, B.Y32, B.w32, B.gid_pk, B.sp_off, k, (int)sh.S_cap, B.cstat, n, B.cself);
    ok = launch_phase2_cos(st, sh.mprec, DM, A);
  } else if (sh.mfma) {
    launch_center(st, sh.mprec, DM, B.Y32, B.w32, B.sp_off, B.cnt, B.csize, k, B.mu, sh.bounds ? B.brec : nullptr);
    A.perm = B.perm;
    A.split = sh.split32;
    ProbeArgs P;
    if (sh.bounds && plan.limit >= 0) P = {X, labels, B.perm, B.brec, n, d};
    ok = launch_pack_mfma(st, sh.mprec, DM, B.Y32, B.w32, B.sp_off, B.cnt, k, B.mu, (int)sh.S_cap, B.Ym, P);
    if (ok && sh.bounds) {
      A.mask = launch_bounds(st, DM, X, n, d, labels, B.perm, B.brec, k, plan.limit, B.bmask);
    }
    ok = ok && launch_phase2_mfma(st, sh.mprec, DM, A, B.mu, B.Ym, mfma_pb_default(sh.mprec, DM));
  } else {
    ok = launch_phase2_valu(st, metric, DM, A);
  }
  if (!ok) return set_error(SILH_E_UNSUPPORTED, "no Phase-2 kernel for this metric and dimension");
  launch_mean(st, B.bpart, (int)ceil_div(n, sh.p2_rows), n, B.mean, sh.split32 ? (int)ceil_div(n, 32) : 0);
  // the status word and the mean come back together: B.status and B.mean are
  // the first two 256-byte slices, so one copy of 264 bytes holds both
  struct {
    int status;
    unsigned char pad[252];
    double mean;
  } back;
  static_assert(sizeof(back) == 264, "status / mean read-back layout");
  if (hipGetLastError() != hipSuccess ||
      hipMemcpyAsync(&back, B.status, sizeof(back), hipMemcpyDeviceToHost, st) != hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess) {
    (void)hipGetLastError();
    return set_error(SILH_E_HIP, "a kernel launch or the read-back failed");
  }
  if (back.status & kStatusLabel) {
    char msg[96];
    std::snprintf(msg, sizeof msg, "a label lies outside [0, %d)", k);
    return set_error(SILH_E_LABEL, msg);
  }
  if (back.status & kStatusEmpty)
    return set_error(SILH_E_K, "fewer than two nonempty clusters; the silhouette needs at least 2");
  if (back.status != 0) return set_error(SILH_E_HIP, "unexpected capacity status");
  if (s_mean_host) *s_mean_host = back.mean;
  return SILH_OK;
}
