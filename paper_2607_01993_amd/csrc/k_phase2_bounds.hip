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
#include "device_common.hpp"
#include "silh_internal.hpp"

namespace silh {

namespace {
constexpr int kHead = 8;  // floats: Wt/|C| (-1: empty cluster), V, slack, E of D, E const, padding
}  // namespace

// floats per cluster record: head, m_j [DM]
size_t bound_rec_floats(int DM) { return (size_t)kHead + DM; }
size_t bound_mask_words(int64_t n, int k) { return (size_t)ceil_div(n, 32) * (size_t)((k + 31) / 32); }

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
        rec[(size_t)j * (kHead + DM) + kHead + c] = mean;
        sh2 = sh * sh;
        n2 = (double)mean * (double)mean;
        g2 = ((double)mean - (double)mv) * ((double)mean - (double)mv);
      }
    } else if (c < DM && rec != nullptr) {
      rec[(size_t)j * (kHead + DM) + kHead + c] = 0.0f;
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
    float* out = rec + (size_t)j * (kHead + DM);
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

// A block takes 64 elements (two mask groups), their rows in LDS, one element
// per lane of each wave; wave w takes cluster pairs as k_p2_cos does.  Up to
// kBndKeep clusters the lower bounds wait in LDS for the smallest upper bound;
// beyond, a first sweep finds that bound and a second one tests against it.
// Waves and kept bounds per row width: the LDS of a block (rows of 64
// elements, kept bounds) leaves at least 16 waves per CU at every width.
// n = 1e6, d = 32, k = 16: 69 us with 4 waves, 77 with 8 and 128 kept; n =
// 5e5, d = 256, k = 16: 512 us with 4 waves (one block per CU), 183 with 8;
// n = 150,001, d = 16, k = 100: 42 us in two sweeps, 32 in one.
template <int DM>
constexpr int kBndWaves = DM == 32 ? 4 : 8;
template <int DM>
constexpr int kBndKeep = DM <= 16 ? 128 : DM == 256 ? 32 : 64;

template <int DM>
__global__ __launch_bounds__((64 * kBndWaves<DM>)) void k_bounds(const float* __restrict__ X, int n, int d,
                                                           const int32_t* __restrict__ labels,
                                                           const int32_t* __restrict__ perm,
                                                           const float* __restrict__ rec, int k,
                                                           uint32_t* __restrict__ mask) {
  constexpr int NW = kBndWaves<DM>, NT = 64 * NW, LD = DM + 4;
  __shared__ __attribute__((aligned(16))) float xs[64 * LD];
  __shared__ float low[kBndKeep<DM>][64];
  __shared__ float um[NW][64];
  __shared__ uint32_t bits[2][128];  // k <= 4096
  __shared__ int rows[64];
  const int row0 = blockIdx.x * 64;
  const int kw = (k + 31) >> 5;
  if (threadIdx.x < 64) {
    const int i = row0 + (int)threadIdx.x < n ? row0 + (int)threadIdx.x : n - 1;
    rows[threadIdx.x] = perm != nullptr ? perm[i] : i;
  }
  for (int q = threadIdx.x; q < 256; q += NT) bits[q >> 7][q & 127] = 0u;
  __syncthreads();
  const bool vec = (d & 3) == 0 && ((uintptr_t)X & 15) == 0;
  if (vec) {
    for (int q = threadIdx.x; q < 64 * (DM / 4); q += NT) {
      const int r = q / (DM / 4), c = (q - r * (DM / 4)) * 4;
      float4 v = float4{0.f, 0.f, 0.f, 0.f};
      if (c < d) v = *(const float4*)(X + (size_t)rows[r] * d + c);
      *(float4*)(xs + r * LD + c) = v;
    }
  } else {
    for (int q = threadIdx.x; q < 64 * DM; q += NT) {
      const int r = q / DM, c = q - r * DM;
      xs[r * LD + c] = c < d ? X[(size_t)rows[r] * d + c] : 0.0f;
    }
  }
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  int own = labels[rows[lane]];
  own = (unsigned)own < (unsigned)k ? own : 0;  // labels are checked before; stay in bounds
  __syncthreads();
  const float* xl = xs + lane * LD;
  constexpr size_t RS = (size_t)kHead + DM;
  // |x - m_j|^2 of two clusters
  auto dist2 = [&](int j, int j2, float (&out)[2]) {
    const float* m0 = rec + (size_t)j * RS + kHead;
    const float* m1 = rec + (size_t)j2 * RS + kHead;
    float a0 = 0.f, a1 = 0.f, b0 = 0.f, b1 = 0.f;
#pragma unroll 4
    for (int c = 0; c < DM; c += 4) {
      const float4 x = *(const float4*)(xl + c);
      float t;
      t = x.x - m0[c]; a0 = fmaf(t, t, a0);
      t = x.y - m0[c + 1]; a1 = fmaf(t, t, a1);
      t = x.z - m0[c + 2]; a0 = fmaf(t, t, a0);
      t = x.w - m0[c + 3]; a1 = fmaf(t, t, a1);
      t = x.x - m1[c]; b0 = fmaf(t, t, b0);
      t = x.y - m1[c + 1]; b1 = fmaf(t, t, b1);
      t = x.z - m1[c + 2]; b0 = fmaf(t, t, b0);
      t = x.w - m1[c + 3]; b1 = fmaf(t, t, b1);
    }
    out[0] = a0 + a1;
    out[1] = b0 + b1;
  };
  float umin = __builtin_inff();
  // sweep 0: upper bounds (and lower bounds kept); sweep 1: the test
  const bool kept = k <= kBndKeep<DM>;
  auto sweep = [&](bool test) {
    for (int j0 = 2 * wave; j0 < k; j0 += 2 * NW) {
      float D2[2];
      dist2(j0, j0 + 1 < k ? j0 + 1 : j0, D2);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int j = j0 + u;
        if (j >= k) break;
        const float* h = rec + (size_t)j * RS;
        const float f = h[0];
        const float D = __builtin_amdgcn_sqrtf(D2[u]);
        const float E = fmaf(h[3], D, h[4]);
        float L = f * (fmaf(D, 1.0f - 0x1p-14f, -h[2]) - E);
        if (f < 0.0f) L = __builtin_inff();  // an empty cluster is never evaluated
        if (!test) {
          const float Dp = D * (1.0f + 0x1p-14f) + h[2];
          const float U = f * (__builtin_amdgcn_sqrtf(fmaf(Dp, Dp, h[1])) * (1.0f + 0x1p-14f) + E);
          if (f >= 0.0f && j != own) umin = fminf(umin, U);
          if (kept) low[j][lane] = L;
        } else if (f >= 0.0f) {
          const uint64_t b = __ballot(!(L > umin));
          if (lane == 0 && (uint32_t)b) atomicOr(&bits[0][j >> 5], 1u << (j & 31));
          if (lane == 32 && (uint32_t)(b >> 32)) atomicOr(&bits[1][j >> 5], 1u << (j & 31));
        }
      }
    }
  };
  sweep(false);
  um[wave][lane] = umin;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NW; ++i) umin = fminf(umin, um[i][lane]);
  if (kept) {
    for (int j = wave; j < k; j += NW) {
      const float f = rec[(size_t)j * RS];
      const uint64_t b = __ballot(f >= 0.0f && !(low[j][lane] > umin));
      if (lane == 0 && (uint32_t)b) atomicOr(&bits[0][j >> 5], 1u << (j & 31));
      if (lane == 32 && (uint32_t)(b >> 32)) atomicOr(&bits[1][j >> 5], 1u << (j & 31));
    }
  } else {
    sweep(true);
  }
  if (wave == 0) atomicOr(&bits[lane >> 5][own >> 5], 1u << (own & 31));
  __syncthreads();
  for (int q = threadIdx.x; q < 2 * kw; q += NT) {
    const int g = q / kw, wd = q - g * kw;
    if (row0 + 32 * g < n) mask[(size_t)(blockIdx.x * 2 + g) * kw + wd] = bits[g][wd];
  }
}

void launch_bounds(hipStream_t st, int DM, const float* X, int n, int d, const int32_t* labels, const int32_t* perm,
                   const float* rec, int k, uint32_t* mask) {
  if (n <= 0) return;
  const dim3 grid((unsigned)ceil_div(n, 64));
#define SILH_BND(D) \
  hipLaunchKernelGGL(k_bounds<D>, grid, dim3(64 * kBndWaves<D>), 0, st, X, n, d, labels, perm, rec, k, mask)
  switch (DM) {
    case 8: SILH_BND(8); break;
    case 16: SILH_BND(16); break;
    case 32: SILH_BND(32); break;
    case 64: SILH_BND(64); break;
    case 128: SILH_BND(128); break;
    default: SILH_BND(256); break;
  }
#undef SILH_BND
}

}  // namespace silh
