// Phase 2 of Algorithm 1 for the cosine distance.
//
// With unit rows x^, y^ and any centre mu_j,
//   1 - x^.y^ = |x~|^2 / 2 + |y~|^2 / 2 - x~.y~,   x~ = x^ - mu_j,  y~ = y^ - mu_j
// (plus 0.5 per zero vector, whose distance to everything is 1).  This is
// affine in the sample row, so the weighted sum over a cluster's sample
//   W_hat_j(x) = sum_q w_q (1 - x^.y^_q)
//              = Wt (|x~|^2 / 2 + u_x) + B - x~.V,
//   Wt = sum w_q,  B = sum w_q (|y~_q|^2 / 2 + u_q),  V = sum w_q y~_q,
// needs the sample once per cluster (k_cos_stats) and one pass of d steps per
// (element, cluster) instead of one per (element, sample row).  What bounds
// it: the vector ALU, n k d steps of 3.5 (bf16) to 4 (fp8) instructions;
// nothing is a matrix product, because x~ is rounded anew around every centre.
// n = 4e6, d = 128, k = 64, t = 512 (S = 38,233): see the figures at
// launch_phase2_cos.
//
// Rounding is that of the per-pair evaluation with the same operands:
//  bf16  x~ and y~ rounded to bf16, products and sums in float32 or wider,
//        norms of the rounded coordinates;
//  fp8   64 x~ and 64 y~ rounded to e4m3 in the product, norms of the
//        unrounded coordinates.  The self pair then is |v|^2 - |v_q|^2, of
//        either sign; it is clamped at 0 by k_cos_self's term.  (Pairs of
//        distinct sampled rows that coincide keep that rounding error, of
//        either sign and of order 1/2 % of |v|^2, unclamped.)
//  fp32  x~ and y~ in float32, everything after that in float64.
// The centre keeps the terms small: for bf16 and fp8 it is the mean of the
// cluster's first 256 sample rows, for fp32 the weighted mean of the sample,
// which makes V vanish but for the rounding of mu, so that W_hat is a sum of
// two non-negative terms and nothing cancels for clusters of near-parallel
// rows.  Rows equal to the centre give exactly 0 (identical points).
#include "device_common.hpp"
#include "silh_internal.hpp"

namespace silh {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

namespace {
constexpr float kFp8Scale = 64.0f;  // |64 v| <= 128 < 448 for unit rows
constexpr int kCenterRows = 256;
constexpr int kStatHead = 64;       // bytes: Wt, B (float64), padding
}  // namespace

// One cluster's record: head, mu [DM] float32 (fp8: times 64), then V as
// float64 [DM] (fp32), three bf16 pieces [3][DM] (bf16) or float32 [DM] (fp8)
size_t cos_stat_bytes(int DM) { return (size_t)kStatHead + (size_t)DM * 12; }

__device__ __forceinline__ float cos_round(int P, float v) {
  if (P == 1) return (float)(__bf16)v;
  if (P == 2) return __builtin_amdgcn_cvt_f32_fp8(__builtin_amdgcn_cvt_pk_fp8_f32(v, 0.0f, 0, false), 0);
  return v;
}

// one block per cluster: columns in chunks of 32, 32 row groups each
template <int P>
__global__ __launch_bounds__(1024) void k_cos_stats(const float* __restrict__ Y32, int DM,
                                                    const float* __restrict__ w, const float* __restrict__ aux,
                                                    const int32_t* __restrict__ sp_off,
                                                    const int32_t* __restrict__ cnt, size_t stride,
                                                    unsigned char* __restrict__ stat) {
  __shared__ double part[32][33];
  __shared__ double wsum[16], bsum[16];
  __shared__ float mus[32];
  __shared__ double wt_all;
  const int j = blockIdx.x;
  const int m = cnt[j], base = sp_off[j];
  const int cc = threadIdx.x & 31, rg = threadIdx.x >> 5;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  unsigned char* rec = stat + (size_t)j * stride;
  float* mu = (float*)(rec + kStatHead);
  double wt = 0.0, b = 0.0;
  for (int r = threadIdx.x; r < m; r += 1024) {
    const double wr = (double)w[base + r];
    wt += wr;
    b += wr * (double)aux[base + r];
  }
  wt = wave_sum_f64(wt);
  if (lane == 0) wsum[wid] = wt;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int i = 0; i < 16; ++i) t += wsum[i];
    wt_all = t;
  }
  __syncthreads();
  // the sum over the 32 row groups of column cc (valid in row group 0)
  auto column = [&](double v) {
    part[rg][cc] = v;
    __syncthreads();
    double t = 0.0;
    if (rg == 0)
      for (int g = 0; g < 32; ++g) t += part[g][cc];
    __syncthreads();
    return t;
  };
  const int mc = P == 0 ? m : (m < kCenterRows ? m : kCenterRows);
  for (int c0 = 0; c0 < DM; c0 += 32) {
    const int c = c0 + cc;
    const bool in = c < DM;
    const float* y = Y32 + (size_t)base * DM + c;
    double s = 0.0;
    if (in) {
#pragma unroll 4
      for (int r = rg; r < mc; r += 32) {
        const double v = (double)y[(size_t)r * DM];
        s += P == 0 ? (double)w[base + r] * v : v;
      }
    }
    s = column(s);
    if (rg == 0) mus[cc] = m > 0 ? (float)(s / (P == 0 ? wt_all : (double)mc)) : 0.0f;
    __syncthreads();
    const float mc1 = mus[cc];
    double V = 0.0;
    if (in) {
#pragma unroll 4
      for (int r = rg; r < m; r += 32) {
        const double wr = (double)w[base + r];
        const float v = y[(size_t)r * DM] - mc1;
        const double q = (double)cos_round(P, P == 2 ? kFp8Scale * v : v);
        const double nv = P == 1 ? q : (double)v;  // fp8: norms of the unrounded coordinates
        V += wr * q;
        b += 0.5 * wr * nv * nv;
      }
    }
    V = column(V);
    if (rg == 0 && in) {
      mu[c] = P == 2 ? kFp8Scale * mc1 : mc1;
      if (P == 0) {
        ((double*)(mu + DM))[c] = V;
      } else if (P == 1) {
        __bf16* o = (__bf16*)(mu + DM);
        const __bf16 h = (__bf16)(float)V;
        const double r1 = V - (double)(float)h;
        const __bf16 md = (__bf16)(float)r1;
        o[c] = h;
        o[DM + c] = md;
        o[2 * DM + c] = (__bf16)(float)(r1 - (double)(float)md);
      } else {
        mu[DM + c] = (float)V;
      }
    }
  }
  b = wave_sum_f64(b);
  if (lane == 0) bsum[wid] = b;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int i = 0; i < 16; ++i) t += bsum[i];
    ((double*)rec)[0] = wt_all;
    ((double*)rec)[1] = t;
  }
}

void launch_cos_stats(hipStream_t st, int prec, int DM, const float* Y32, const float* w, const float* aux,
                      const int32_t* sp_off, const int32_t* cnt, int k, unsigned char* stat) {
  const size_t stride = cos_stat_bytes(DM);
#define SILH_CS(P) \
  hipLaunchKernelGGL(k_cos_stats<P>, dim3(k), dim3(1024), 0, st, Y32, DM, w, aux, sp_off, cnt, stride, stat)
  if (prec == 1)
    SILH_CS(1);
  else if (prec == 2)
    SILH_CS(2);
  else
    SILH_CS(0);
#undef SILH_CS
}

// fp8: what the clamp at 0 adds to the self pair of each sampled element,
// w (max(0, c) - c) with c = |v|^2 - |v_q|^2, into self[element id] (the
// other elements' entries are 0 before); one wave per packed row
__global__ __launch_bounds__(256) void k_cos_self(const float* __restrict__ Y32, int DM, const float* __restrict__ w,
                                                  const int32_t* __restrict__ gid_pk,
                                                  const int32_t* __restrict__ sp_off, int k, int cap,
                                                  const unsigned char* __restrict__ stat, size_t stride,
                                                  float* __restrict__ self) {
  const int s = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & (kWave - 1);
  if (s >= cap || s >= sp_off[k]) return;
  const int g = gid_pk[s];
  if (g < 0) return;  // padding, or a zero row (its self pair is 1)
  int lo = 0, hi = k;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (sp_off[mid] <= s) lo = mid; else hi = mid;
  }
  const float* mu = (const float*)(stat + (size_t)lo * stride + kStatHead);
  double c = 0.0;
  for (int i = lane; i < DM; i += kWave) {
    const float v = kFp8Scale * Y32[(size_t)s * DM + i] - mu[i];
    const float q = cos_round(2, v);
    c += (double)v * (double)v - (double)q * (double)q;
  }
  c = wave_sum_f64(c);
  if (lane == 0 && c < 0.0) self[g] = (float)(-(double)w[s] * c * (1.0 / ((double)kFp8Scale * kFp8Scale)));
}

void launch_cos_self(hipStream_t st, int DM, const float* Y32, const float* w, const int32_t* gid_pk,
                     const int32_t* sp_off, int k, int cap, const unsigned char* stat, int n, float* self) {
  launch_fill_i32(st, (int32_t*)self, n, 0);
  if (cap > 0)
    hipLaunchKernelGGL(k_cos_self, dim3((int)ceil_div(cap, 4)), dim3(256), 0, st, Y32, DM, w, gid_pk, sp_off, k, cap,
                       stat, cos_stat_bytes(DM), self);
}

// A block takes kCosRows elements, one per lane of each of its NW waves,
// their unit rows in LDS (rows padded by 16 bytes, so the lanes' 16-byte reads
// fall in distinct banks); wave w takes the cluster pairs 2w, 2w + 2 NW, ...,
// whose records are wave-uniform and come in by scalar loads.  Two clusters
// share each read of the row.
template <int P, int DM>
constexpr int kCosWaves = DM >= 128 ? 8 : 4;


template <int P, int DM>
__global__ __launch_bounds__((64 * kCosWaves<P, DM>)) void k_p2_cos(
    const float* __restrict__ X, int n, int d, const int32_t* __restrict__ labels,
    const float* __restrict__ rn, const unsigned char* __restrict__ stat, const int32_t* __restrict__ csize, int k,
    float* __restrict__ a_out, float* __restrict__ b_out, float* __restrict__ s_out, float* __restrict__ What,
    double* __restrict__ bpart, const float* __restrict__ self, const int32_t* __restrict__ egid) {
  constexpr int NW = kCosWaves<P, DM>, NT = 64 * NW, LD = DM + 4;
  constexpr size_t kStride = (size_t)kStatHead + (size_t)DM * 12;
  constexpr float S1 = P == 2 ? kFp8Scale : 1.0f;
  static_assert(kCosRows == kWave, "one element per lane");
  __shared__ __attribute__((aligned(16))) float xs[kCosRows * LD];
  __shared__ double sh_own[kWave], sh_num[NW][kWave], sh_den[NW][kWave];
  const int row0 = blockIdx.x * kCosRows;
  const int nr = n - row0 < kCosRows ? n - row0 : kCosRows;
  // unit rows (times 64 for fp8: a power of two, so x~ is the same times 64),
  // zero past d and past n
  const bool vec = (d & 3) == 0 && ((uintptr_t)X & 15) == 0;
  if (vec) {
    for (int q = threadIdx.x; q < kCosRows * (DM / 4); q += NT) {
      const int r = q / (DM / 4), c = (q - r * (DM / 4)) * 4;
      float4 v = float4{0.f, 0.f, 0.f, 0.f};
      if (r < nr && c < d) {
        v = *(const float4*)(X + (size_t)(row0 + r) * d + c);
        const float f = rn[row0 + r];
        v = float4{v.x * f * S1, v.y * f * S1, v.z * f * S1, v.w * f * S1};
      }
      *(float4*)(xs + r * LD + c) = v;
    }
  } else {
    for (int q = threadIdx.x; q < kCosRows * DM; q += NT) {
      const int r = q / DM, c = q - r * DM;
      xs[r * LD + c] = r < nr && c < d ? X[(size_t)(row0 + r) * d + c] * rn[row0 + r] * S1 : 0.0f;
    }
  }
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int e = row0 + lane, er = e < n ? e : n - 1;
  int own = labels[er];
  own = (unsigned)own < (unsigned)k ? own : 0;  // labels are checked before; stay in bounds
  const double ux = rn[er] > 0.f ? 0.0 : 0.5;
  const double selfv = P == 2 ? (double)self[egid != nullptr ? egid[er] : er] : 0.0;
  if (wave == 0) sh_own[lane] = 0.0;
  __syncthreads();
  const float* xl = xs + lane * LD;
  double bnum = 1.0, bden = 0.0;
  for (int j0 = 2 * wave; j0 < k; j0 += 2 * NW) {
    double W2[2];
    const unsigned char* rec[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) rec[u] = stat + (size_t)(j0 + u < k ? j0 + u : j0) * kStride;
    if constexpr (P == 0) {
      double nx[2] = {0.0, 0.0}, dt[2] = {0.0, 0.0};
#pragma unroll 2
      for (int c = 0; c < DM; c += 4) {
        const float4 x4 = *(const float4*)(xl + c);
        const float x[4] = {x4.x, x4.y, x4.z, x4.w};
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const float* mu = (const float*)(rec[u] + kStatHead);
          const double* V = (const double*)(mu + DM);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const double v = (double)(x[i] - mu[c + i]);
            nx[u] = fma(v, v, nx[u]);
            dt[u] = fma(v, V[c + i], dt[u]);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const double* hd = (const double*)rec[u];
        W2[u] = fma(hd[0], fma(0.5, nx[u], ux), hd[1]) - dt[u];
      }
    } else if constexpr (P == 1) {
      // two float32 chains per sum (even and odd 4-coordinate steps)
      float nx[2][2] = {}, dt[2][2] = {};
#pragma unroll 4
      for (int c = 0; c < DM; c += 4) {
        const int h = (c >> 2) & 1;
        const float4 x4 = *(const float4*)(xl + c);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const float* mu = (const float*)(rec[u] + kStatHead);
          const bf16x2* V = (const bf16x2*)(mu + DM);
          const f32x2 v0 = {x4.x - mu[c], x4.y - mu[c + 1]}, v1 = {x4.z - mu[c + 2], x4.w - mu[c + 3]};
          const bf16x2 q0 = __builtin_convertvector(v0, bf16x2), q1 = __builtin_convertvector(v1, bf16x2);
          nx[u][h] = __builtin_amdgcn_fdot2_f32_bf16(q0, q0, nx[u][h], false);
          nx[u][h] = __builtin_amdgcn_fdot2_f32_bf16(q1, q1, nx[u][h], false);
#pragma unroll
          for (int p = 0; p < 3; ++p) {
            dt[u][h] = __builtin_amdgcn_fdot2_f32_bf16(q0, V[p * (DM / 2) + c / 2], dt[u][h], false);
            dt[u][h] = __builtin_amdgcn_fdot2_f32_bf16(q1, V[p * (DM / 2) + c / 2 + 1], dt[u][h], false);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const double* hd = (const double*)rec[u];
        const double nn = (double)nx[u][0] + (double)nx[u][1];
        W2[u] = fma(hd[0], fma(0.5, nn, ux), hd[1]) - ((double)dt[u][0] + (double)dt[u][1]);
      }
    } else {
      float nx[2][2] = {}, dt[2][2] = {};
#pragma unroll 4
      for (int c = 0; c < DM; c += 4) {
        const int h = (c >> 2) & 1;
        const float4 x4 = *(const float4*)(xl + c);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const float* mu = (const float*)(rec[u] + kStatHead);  // times 64, as x
          const float* V = mu + DM;
          const float v[4] = {x4.x - mu[c], x4.y - mu[c + 1], x4.z - mu[c + 2], x4.w - mu[c + 3]};
          int pk = __builtin_amdgcn_cvt_pk_fp8_f32(v[0], v[1], 0, false);
          pk = __builtin_amdgcn_cvt_pk_fp8_f32(v[2], v[3], pk, true);
          const f32x2 q0 = __builtin_amdgcn_cvt_pk_f32_fp8(pk, false), q1 = __builtin_amdgcn_cvt_pk_f32_fp8(pk, true);
          const float q[4] = {q0.x, q0.y, q1.x, q1.y};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            nx[u][h] = fmaf(v[i], v[i], nx[u][h]);
            dt[u][h] = fmaf(q[i], V[c + i], dt[u][h]);
          }
        }
      }
      constexpr double IS2 = 1.0 / ((double)kFp8Scale * kFp8Scale);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const double* hd = (const double*)rec[u];
        const double nn = ((double)nx[u][0] + (double)nx[u][1]) * IS2;
        W2[u] = fma(hd[0], fma(0.5, nn, ux), hd[1]) - ((double)dt[u][0] + (double)dt[u][1]) * IS2;
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int j = j0 + u;
      if (j >= k) break;
      // a sum of distances: the rounding of the last subtraction may leave a
      // value below 0; an element that is not finite has sums of 0
      double W = W2[u];
      if (P == 2 && j == own) W += selfv;
      W = W > 0.0 ? W : 0.0;
      if (What != nullptr && e < n) What[(size_t)e * k + j] = (float)W;
      const int sz = csize[j];
      const double dsz = (double)sz;
      if (j == own) {
        sh_own[lane] = W;  // one wave's clusters hold the element's own
      } else if (sz > 0 && W * bden < bnum * dsz) {
        bnum = W;
        bden = dsz;
      }
    }
  }
  sh_num[wave][lane] = bnum;
  sh_den[wave][lane] = bden;
  __syncthreads();
  if (wave != 0) return;
#pragma unroll
  for (int i = 1; i < NW; ++i) {
    const double num = sh_num[i][lane], den = sh_den[i][lane];
    if (den > 0.0 && num * bden < bnum * den) {
      bnum = num;
      bden = den;
    }
  }
  const int szo = csize[own];
  const double a = szo > 1 ? sh_own[lane] / (double)(szo - 1) : 0.0;
  const double b = bden > 0.0 ? bnum / bden : __builtin_inf();
  const double mx = a > b ? a : b;
  const double s = (szo > 1 && mx > 0.0) ? (b - a) / mx : 0.0;
  if (e < n) {
    if (a_out) a_out[e] = (float)a;
    if (b_out) b_out[e] = (float)b;
    if (s_out) s_out[e] = (float)s;
  }
  const double tot = wave_sum_f64(e < n ? s : 0.0);
  if (lane == 0) bpart[blockIdx.x] = tot;
}

template <int P, int DM>
static void launch_cos_one(hipStream_t st, const P2Args& A) {
  hipLaunchKernelGGL((k_p2_cos<P, DM>), dim3((int)ceil_div(A.n, kCosRows)), dim3(64 * kCosWaves<P, DM>), 0, st, A.X,
                     A.n, A.d, A.labels, A.rn, A.cstat, A.csize, A.k, A.a, A.b, A.s, A.What, A.bpart, A.cself, A.egid);
}

template <int P>
static bool launch_cos_prec(hipStream_t st, int DM, const P2Args& A) {
  switch (DM) {
    case 8: launch_cos_one<P, 8>(st, A); return true;
    case 16: launch_cos_one<P, 16>(st, A); return true;
    case 32: launch_cos_one<P, 32>(st, A); return true;
    case 64: launch_cos_one<P, 64>(st, A); return true;
    case 128: launch_cos_one<P, 128>(st, A); return true;
    case 256: launch_cos_one<P, 256>(st, A); return true;
    default: return false;
  }
}

// Phase 2 measured, per pair (matrix cores) -> collapsed: n = 4e6, d = 128,
// k = 64, S = 38,233, bf16 42.5 -> 3.67 ms (3.3e10 coordinate steps at 8.9e12
// a second); n = 1e6, d = 100, k = 48, S = 15,000, fp8 4.44 -> 0.80 ms.  The
// collapsed sums win at every S above a few rows per cluster, so there is no
// rule and no other path.
static bool launch_cos_rows(hipStream_t st, int prec, int DM, const P2Args& A) {
  if (prec == 1) return launch_cos_prec<1>(st, DM, A);
  if (prec == 2) return launch_cos_prec<2>(st, DM, A);
  return launch_cos_prec<0>(st, DM, A);
}

// pieces: as tab_plan's, about 1 ms of coordinate steps each (a block's rows
// do not depend on the others': the same results)
constexpr int64_t kPieceSteps = (int64_t)1 << 33;

bool launch_phase2_cos(hipStream_t st, int prec, int DM, const P2Args& A, bool pieces) {
  int64_t rows = A.n;
  if (pieces) {
    rows = kPieceSteps / ((int64_t)A.k * DM) / kCosRows * kCosRows;
    rows = rows < kCosRows ? kCosRows : rows;
  }
  for (int64_t i0 = 0; i0 < A.n; i0 += rows) {
    P2Args B = A;
    B.n = (int)(A.n - i0 < rows ? A.n - i0 : rows);
    B.X += i0 * A.d;
    B.labels += i0;
    B.rn += i0;
    if (B.egid)
      B.egid += i0;
    else if (B.cself)
      B.cself += i0;
    if (B.a) B.a += i0;
    if (B.b) B.b += i0;
    if (B.s) B.s += i0;
    if (B.What) B.What += i0 * A.k;
    B.bpart += i0 / kCosRows;
    if (!launch_cos_rows(st, prec, DM, B)) return false;
    if (i0 + rows < A.n && hipStreamSynchronize(st) != hipSuccess) return true;  // (the next call reports it)
  }
  return true;
}

}  // namespace silh
