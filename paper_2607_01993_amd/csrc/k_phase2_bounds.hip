// Which clusters an element's Euclidean scores need.
//
// silh_scores takes W_hat of the element's own cluster (a_hat) and the smallest
// W_hat_j / |C_j| over the others (b_hat).  With m_j the weighted mean of
// cluster j's sample, Wt_j the sum of its weights and V_j its weighted mean of
// |y - m_j|^2, the sum of distances lies between
//   Wt_j |x - m_j|  <=  sum_q w_q |x - y_q|  <=  Wt_j sqrt(|x - m_j|^2 + V_j)
// (convexity of the norm; Cauchy-Schwarz), d steps per (element, cluster) for
// both.  A cluster whose lower bound exceeds another's upper bound cannot be
// the smallest: its sum is not evaluated.  The bounds are widened by more
// than the Phase-2 kernel's own rounding error (below), so a_hat, b_hat, s_hat
// and the mean are those of evaluating every cluster, bit for bit.
//
// Widening.  With x~ = x - mu_j, y~ = y - mu_j (mu_j the kernel's centre, g_j =
// |m_j - mu_j|, D = |x - m_j|).  bf16 operands have eight significant bits: each
// coordinate moves by up to 2^-8 of itself (257 -> 256), each distance by at
// most 2^-8 (|x~| + |y~|).  The float32 expansion, 272 terms at most, each
// addition 2^-23 of the terms' sum (|x~| + |y~|)^2, errs by 2^-16 (|x~| + |y~|)^2 / d
// more; pairs with c < 6 tau |x~|^2 (or |y~|^2, by the layout) are evaluated
// directly, so d is at least 0.153 of that norm r, the other at most r + d, and
// the error at most 2^-15 (15 r + d).  Together below
// 2^-8 (1.12 |x~| + 1.12 |y~| + 0.03 d), and with |x~| <= D + g, the mean of |y~| at
// most sqrt(V) + g, the mean of d at most D + sqrt(V):
//   E = Wt 2^-8 (1.33 D + 1.2 sqrt(V) + 2.4 g).
// float32 operands: d is at least 0.43 |x~| there, the expansion's error at most
// 2^-16 (7 |x~| + d) (132 terms; of three pieces a coordinate, 64 terms of full
// size), covered by the same expression with 2^-13.  The float32 rounding of
// m_j, of D (at most 256 steps) and of the sums below is covered by relative
// slacks of 2^-14 and an absolute one of 2^-22 |m_j|.
//
// The groups of 32 elements that a Phase-2 wave holds share a mask, the union
// over the group, so elements go in cluster order (the index's permutation):
// a group then has one own cluster (mostly) and nearby ones.
#include "bounds_block.hpp"

namespace silh {

// the clusters' records, then the probe's counts
size_t bound_rec_floats(int DM, int k) { return (size_t)k * (kBoundRec + DM) + kBoundProbe; }
size_t bound_mask_words(int64_t n, int k) {
  return kBoundHead + (size_t)ceil_div(n, 32) * (size_t)((k + 31) / 32);
}

// The clusters' centres mu_j (the mean of the first kCenterRows sample rows;
// any point of the cluster would do, the mean keeps the centred operands
// smallest), the squared radii's zeros, and with rec non-null the bound
// records, in one pass over the packed sample.  One block per cluster; a
// thread holds four columns and takes every G-th row, sums in float64 about
// the cluster's first row.  (k = 16, d = 256, S = 4,324: the two passes in
// chunks of 32 columns that this replaces took 27 and 28 us.)
constexpr int kCenterRows = 256;

__global__ __launch_bounds__(1024) void k_center(const float* __restrict__ Y32, int DM, int KP,
                                                 const float* __restrict__ w,
                                                 const int32_t* __restrict__ sp_off,
                                                 const int32_t* __restrict__ cnt,
                                                 const int32_t* __restrict__ csize, float eta,
                                                 float* __restrict__ mu, float* __restrict__ rec) {
  __shared__ double part[16][256];
  __shared__ double red[16][2];
  __shared__ double fin[4][3];
  __shared__ double wt_all, q_all;
  const int j = blockIdx.x;
  const int m = cnt[j], base = sp_off[j], sz = csize[j];
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  const int L = DM >> 2, G = 1024 / L;  // column quads (a power of two, at most 64), row groups
  const int cl = threadIdx.x & (L - 1), rg = threadIdx.x / L;
  const int mc = m < kCenterRows ? m : kCenterRows;
  const float* y = Y32 + (size_t)base * DM + 4 * cl;
  float4 y0 = float4{0.f, 0.f, 0.f, 0.f};
  if (m > 0) y0 = *(const float4*)y;
  double s1[4] = {}, sw[4] = {}, q = 0.0, wt = 0.0;
#pragma unroll 4
  for (int r = rg; r < m; r += G) {
    const float4 v = *(const float4*)(y + (size_t)r * DM);
    const double wr = (double)w[base + r];
    const bool in = r < mc;  // (a product with 0 would bring a later row's Inf or NaN into the centre)
    const double dv[4] = {(double)v.x - (double)y0.x, (double)v.y - (double)y0.y, (double)v.z - (double)y0.z,
                          (double)v.w - (double)y0.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s1[e] += in ? dv[e] : 0.0;
      sw[e] += wr * dv[e];
      q += wr * dv[e] * dv[e];
    }
    if (cl == 0) wt += wr;
  }
  // the sum of a column over the row groups: lanes of the wave that share its
  // quad, then the 16 waves (valid in thread c < DM for column c)
  auto columns = [&](double (&v)[4]) {
    for (int o = L; o < kWave; o <<= 1)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += __shfl_xor(v[e], o, kWave);
    __syncthreads();
    if (lane < L)
#pragma unroll
      for (int e = 0; e < 4; ++e) part[wid][4 * cl + e] = v[e];
    __syncthreads();
    double t = 0.0;
    if ((int)threadIdx.x < DM)
      for (int i = 0; i < 16; ++i) t += part[i][threadIdx.x];
    return t;
  };
  const double c1 = columns(s1);
  const double cw = columns(sw);
  wt = wave_sum_f64(wt);
  q = wave_sum_f64(q);
  if (lane == 0) {
    red[wid][0] = wt;
    red[wid][1] = q;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = 0.0, b = 0.0;
    for (int i = 0; i < 16; ++i) {
      a += red[i][0];
      b += red[i][1];
    }
    wt_all = a;
    q_all = b;
    mu[(size_t)gridDim.x * KP + j] = 0.0f;  // the squared radius, whose maximum the packing takes
  }
  __syncthreads();
  const int c = threadIdx.x;
  const double wa = wt_all;
  double sh2 = 0.0, n2 = 0.0, g2 = 0.0;  // |m - y0|^2, |m|^2, |m - mu|^2
  if (c < KP) {
    float mv = 0.0f;
    if (c < DM && m > 0) {
      const double yc = (double)Y32[(size_t)base * DM + c];
      mv = (float)(yc + c1 / (double)mc);
      if (rec != nullptr) {
        const double sh = wa > 0.0 ? cw / wa : 0.0;
        const float mean = (float)(yc + sh);
        rec[(size_t)j * (kBoundRec + DM) + kBoundRec + c] = mean;
        sh2 = sh * sh;
        n2 = (double)mean * (double)mean;
        g2 = ((double)mean - (double)mv) * ((double)mean - (double)mv);
      }
    } else if (c < DM && rec != nullptr) {
      rec[(size_t)j * (kBoundRec + DM) + kBoundRec + c] = 0.0f;
    }
    mu[(size_t)j * KP + c] = mv;
  }
  if (rec == nullptr) return;  // block-uniform
  if (wid < 4) {
    sh2 = wave_sum_f64(sh2);
    n2 = wave_sum_f64(n2);
    g2 = wave_sum_f64(g2);
    if (lane == 0) {
      fin[wid][0] = sh2;
      fin[wid][1] = n2;
      fin[wid][2] = g2;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    sh2 = fin[0][0] + fin[1][0] + fin[2][0] + fin[3][0];
    n2 = fin[0][1] + fin[1][1] + fin[2][1] + fin[3][1];
    g2 = fin[0][2] + fin[1][2] + fin[2][2] + fin[3][2];
    const double qm = wa > 0.0 ? q_all / wa : 0.0;
    double V = qm - sh2;
    V = (V > 0.0 ? V : 0.0) + 1e-12 * qm;  // (the difference's rounding)
    float* out = rec + (size_t)j * (kBoundRec + DM);
    out[0] = sz > 0 ? (float)(wa / (double)sz) : -1.0f;
    out[1] = (float)(V * (1.0 + 0x1p-14));
    out[2] = (float)(sqrt(n2) * 0x1p-22);
    out[3] = 1.33f * eta;
    out[4] = (float)((double)eta * (1.2 * sqrt(V) + 2.4 * sqrt(g2)));
    out[5] = out[6] = out[7] = 0.0f;
  }
}

void launch_center(hipStream_t st, int prec, int DM, const float* Y32, const float* w, const int32_t* sp_off,
                   const int32_t* cnt, const int32_t* csize, int k, float* mu, float* rec) {
  hipLaunchKernelGGL(k_center, dim3(k), dim3(1024), 0, st, Y32, DM, mfma_kp(prec, DM), w, sp_off, cnt, csize,
                     prec == 1 ? 0x1p-8f : 0x1p-13f, mu, rec);
}

// The masks.  `counts` (null without a probe: scalar loads): the block returns
// at once where the probe's counts exceed the limit; the first block says
// which in head[kBoundFlag].
template <int DM>
__global__ __launch_bounds__((64 * kBndWaves<DM>)) void k_bounds(const float* __restrict__ X, int n, int d,
                                                           const int32_t* __restrict__ labels,
                                                           const int32_t* __restrict__ perm,
                                                           const float* __restrict__ rec, int k, int limit,
                                                           const uint32_t* __restrict__ counts,
                                                           uint32_t* __restrict__ head) {
  bounds_block<DM, kBndWaves<DM>, false>(X, n, d, labels, perm, rec, k, (int)blockIdx.x * 64, head + kBoundHead, [&] {
    bool skip = false;
    if (counts != nullptr) {
      int c = 0;
#pragma unroll
      for (int i = 0; i < kBoundProbe; ++i) c += (int)counts[i];
      skip = c > limit;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) head[kBoundFlag] = skip ? 1u : 0u;
    return skip;
  });
}

const uint32_t* launch_bounds(hipStream_t st, int DM, const float* X, int n, int d, const int32_t* labels,
                              const int32_t* perm, const float* rec, int k, int limit, uint32_t* buf) {
  if (n <= 0) return buf + kBoundHead;
  const dim3 grid((unsigned)ceil_div(n, 64));
  const uint32_t* counts = limit >= 0 ? (const uint32_t*)(rec + (size_t)k * (kBoundRec + DM)) : nullptr;
#define SILH_BND(D)                                                                                             \
  hipLaunchKernelGGL(k_bounds<D>, grid, dim3(64 * kBndWaves<D>), 0, st, X, n, d, labels, perm, rec, k, limit, \
                     counts, buf)
  switch (DM) {
    case 8: SILH_BND(8); break;
    case 16: SILH_BND(16); break;
    case 32: SILH_BND(32); break;
    case 64: SILH_BND(64); break;
    case 128: SILH_BND(128); break;
    default: SILH_BND(256); break;
  }
#undef SILH_BND
  return buf + kBoundHead;
}

// What the bounds cost against what they can save, in microseconds at the rates
// measured for both (bf16 and float32 requests of n = 20,000 to 400,000, k = 3
// to 64, 32 to 512 sample rows a cluster, d = 16, 64, 256, clusters that touch
// and labels that have nothing to do with the data).  A pair of Phase 2 takes p,
// a cluster as much as 64 rows more; the bounds take an element's row again and
// a share a cluster.  Two of k clusters are needed at least.  From 65,536
// elements on (below, the chip is not full, and both sides take about as long
// as there) the probe finds how many are, where its own chain (k / 8 cluster
// pairs) is hidden by the packing or small next to the bounds; without it 0.6
// of the most is expected.  Without -> with the bounds: n = 400,000, m = 128,
// cells, d = 16 k = 5 232 -> 256 us, k = 64 803 -> 462; d = 256 k = 3 512 -> 678,
// k = 64 3,558 -> 2,980; n = 20,000, m = 512, d = 256 k = 3 253 -> 270, k = 8 492 -> 453;
// random labels d = 64 k = 16 436 -> 498.
BoundPlan bound_plan(int prec, int DM, int64_t n, int k, int64_t S) {
  BoundPlan b;
  if (k <= 2 || n * S < ((int64_t)1 << 24)) return b;
  const double nn = n < 65536 ? 65536.0 : (double)n;
  const double p = prec == 1 ? 1.8e-7 + 2.2e-9 * DM : 3e-7 + 9e-9 * DM;
  const double sums = nn * ((double)S + 64.0 * (double)k) * p;
  const double cost = 1.1 * nn * (3e-5 + 1.1e-6 * DM + (double)k * (1e-6 + 4e-8 * DM));
  const double chain = (double)k / 8.0 * (1.5 + 0.04 * DM);
  const double most = 1.0 - 2.0 / (double)k;
  const bool probe = n >= 65536 && (chain <= 8.0 || chain < 0.3 * cost);
  b.use = (probe ? 1.0 : 0.6) * most * sums > 1.5 * cost + 20.0;
  if (b.use && probe) b.limit = (int)((1.0 - cost / sums) * (double)k * 2.0 * kBoundProbe);
  return b;
}

}  // namespace silh
