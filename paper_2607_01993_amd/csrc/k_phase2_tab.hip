// Phase 2 of Algorithm 1 for Manhattan and Canberra by per-coordinate tables.
//
// Both distances are sums over coordinates, so a cluster's weighted sum is
//   W_hat_j(x) = sum_c f_{j,c}(x_c),   f_{j,c}(t) = sum_q w_q delta(t, y_{q,c}),
// delta(t, y) = |t - y| (Manhattan) or |t - y| / (|t| + |y|) (Canberra, 0/0 = 0):
// functions of one variable, whose only kinks are the sample's own values.  A
// table per (cluster, coordinate) holds f at those values (the knots); an
// element finds its interval (a lookup by a uniform grid over the knots, then
// a few search steps, all in LDS) and interpolates, about 30 instructions per
// (element, cluster, coordinate) whatever the number of sample rows, against 2
// (Manhattan) or 4.6 (Canberra) per row.  What bounds it: the vector ALU and
// the LDS reads.
//
//  Manhattan  f is linear between knots: with a = y_{i+1} - t, b = t - y_i,
//             f = a g_i + b h_i, g = f_i / gap, h = f_{i+1} / gap, both terms
//             >= 0; outside the knots f adds Wt |t - nearest knot|.
//  Canberra   f is smooth between knots, with poles at the negatives of the
//             values: cubic between knots, f = a g + b h + a b (c0 + c1 b), the
//             residual of the linear part interpolated at the quarter points.
//             The knots are refined until the cubic's error stays below the
//             rounding of float32 (kCanbStep below).  Opposite signs are
//             at distance 1, so each sign of t has its own smooth part; beyond
//             Y, twice the largest magnitude of a sign, the table runs over
//             z = Y (2 - Y / |t|), which maps |t| -> infinity to 2 Y (up to Y z
//             is t itself: f can be small next to the sample, and the map's
//             rounding would not be).
//             At t = 0 f jumps to the weights of the nonzero values
//             alone: a record of its own (Wt less the zeros' weights would
//             leave their rounding where the sum is small or 0).
//
// Precision: table values from float64 sums (Canberra: of float32 terms good
// to an ulp), kept, interpolated and added up in float64; only the cubic's
// residual, below a thousandth of f, is float32.  Every term of the linear part
// is >= 0 and the knots are exact, so results are relative to f itself: rows
// equal to all of a cluster's values are at distance exactly 0.
// A table is not used (its rows are summed directly, in float32 as by k_p2_valu)
// where a value is not finite, Canberra's where a magnitude lies outside [2^-30,
// 2^30] (0 is fine; Manhattan's up to 2^126), or the refinement outgrows the
// table; the elements' values are arbitrary (Canberra: a wave with one past
// 2^62 or not finite sums directly too).
//
// Clusters of more than kTabRows sample rows take several tables (chunks).
#include <float.h>

#include "device_common.hpp"
#include "silh_internal.hpp"

namespace silh {

namespace {
constexpr int kTabRows = 1024;           // sample rows per table at most
constexpr int kTabExtra = 512;           // knots beyond twice the rows
constexpr int kTabKnots = 2 * kTabRows + kTabExtra;
constexpr int kTabMost = kTabKnots - (kTabRows + 8);  // Canberra (base knots wait behind them)
constexpr int kBuildT = 256, kEvalT = 256;
// The lookup: grid cell b = (z - z0) NB / (z1 - z0) starts at the last knot of an
// earlier cell; L steps of 2^(L-1), .., 1 knots then reach any knot of the cell.
// Tables with a cell of more than 2^kTabSteps knots are searched in halves.
constexpr int kTabCells = 512, kTabSteps = 6, kTabPad = 1 << kTabSteps;
constexpr float kTabMin = 0x1p-30f, kTabMax = 0x1p30f;
constexpr float kManhMax = 0x1p126f;  // (differences of two stay finite)
constexpr float kPairMax = 0x1p46f;   // Canberra summed directly in pairs of rows: w n d <= 2^124
// Canberra: knots in steps of at most kCanbStep (f / Wt)^(1/4) of ln(t + u), u
// the smallest magnitude of the sign, f the smaller of the segment's ends but
// no less than kCanbFloor Wt: where f starts from 0 it reaches s Wt / 2 within
// the step, and the error, which vanishes at the knots, is relative to that.  With gap = s (t + u) <= s (t + y) the
// cubic through the ends and quarter points errs by at most
// max |tau (1 - tau) (tau - 1/4)(tau - 3/4)| gap^4 sum 2 w y / (t + y)^5
// <= s^4 / 64 sum 2 w y / (t + y) <= s^4 Wt / 32: 2^-24 f at half a step's
// typical y / (t + y), and zero at four points of the interval.
constexpr float kCanbStep = 0.04f, kCanbFloor = 0.0054f;
constexpr size_t kTabGroupBytes = (size_t)512 << 20;  // tables held at once
constexpr int64_t kPieceEvals = (int64_t)1 << 29;     // about 1 ms of evaluations (tab_plan's pieces)
constexpr int64_t kTabWork = (int64_t)1 << 26;        // float64 sums held at once
}  // namespace

// one (chunk, coordinate) table's head
struct TabHead {
  int K;           // knots; 0: sum directly, -1: and a value past kPairMax or not finite
  int L;           // steps within a cell
  float inv, off;  // cell = z inv + off
  float lo, hi;    // Manhattan: first and last knot; Canberra: minus / plus twice the largest magnitude of
                   // the negative / positive values (1 if none)
  float Wt;        // Manhattan: sum of the weights
  float zero;      // Canberra: the knot past the record for zeros, 0 if the sample has none
};

// the grid cell of z (the same instructions when the table is built and read)
__device__ __forceinline__ int tab_cell(float z, float inv, float off) {
  const int b = (int)fmaxf(fmaf(z, inv, off), 0.0f);
  return b < kTabCells ? b : kTabCells - 1;
}

// ----------------------------------------------------------------------------
// chunks: cluster j's sample rows in ceil(cnt / kTabRows) equal parts; chunk =
// (cluster, first packed row, rows, 1 if the cluster's first); cfirst[j] the
// cluster's first chunk, cfirst[k] their number
// ----------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void k_tab_chunks(const int32_t* __restrict__ sp_off,
                                                     const int32_t* __restrict__ cnt, int k, int cap,
                                                     int4* __restrict__ chunk, int32_t* __restrict__ cfirst) {
  __shared__ int32_t part[1024];
  const int per = (k + 1023) / 1024;
  const int j0 = threadIdx.x * per, j1 = j0 + per < k ? j0 + per : k;
  int s = 0;
  for (int j = j0; j < j1; ++j) s += (cnt[j] + kTabRows - 1) / kTabRows;
  part[threadIdx.x] = s;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const int v = (int)threadIdx.x >= o ? part[threadIdx.x - o] : 0;
    __syncthreads();
    part[threadIdx.x] += v;
    __syncthreads();
  }
  int at = threadIdx.x ? part[threadIdx.x - 1] : 0;
  for (int j = j0; j < j1; ++j) {
    const int m = cnt[j], nc = (m + kTabRows - 1) / kTabRows;
    cfirst[j] = at < cap ? at : cap;
    const int rows = nc > 0 ? (m + nc - 1) / nc : 0;
    for (int q = 0; q < nc; ++q, ++at)
      if (at < cap) chunk[at] = int4{j, sp_off[j] + q * rows, q + 1 < nc ? rows : m - q * rows, q == 0 ? 1 : 0};
  }
  if (threadIdx.x == 1023) cfirst[k] = part[1023] < cap ? part[1023] : cap;
}

// A chunk's tables start at knot (2 row + kTabExtra chunk) past the group's
// first chunk's, times the coordinates
__device__ __forceinline__ size_t tab_base(const int4* __restrict__ chunk, int q, int q0) {
  return (size_t)(2 * (chunk[q].y - chunk[q0].y) + kTabExtra * (q - q0));
}

// |t - y| / (t + y) for t, y >= 0 not both 0, to about an ulp
__device__ __forceinline__ float canb_term(float num, float den) {
  const float r = __builtin_amdgcn_rcpf(den);
  const float v = num * r;
  return fmaf(fmaf(-den, v, num), r, v);
}

// ----------------------------------------------------------------------------
// one block per (coordinate, chunk of the group): sort the values, place the
// knots, sum f at the knots (Canberra: and at the quarter points)
// ----------------------------------------------------------------------------
template <int M>
__global__ __launch_bounds__(kBuildT) void k_tab_build(const float* __restrict__ Y32, int DM, int d,
                                                       const float* __restrict__ w,
                                                       const int4* __restrict__ chunk,
                                                       const int32_t* __restrict__ cfirst, int k, int q0,
                                                       TabHead* __restrict__ head, float* __restrict__ tabY,
                                                       double* __restrict__ tabG, float2* __restrict__ tabC,
                                                       uint16_t* __restrict__ tabL) {
  __shared__ float ys[kTabRows], ws[kTabRows];
  __shared__ float kn[kTabKnots];
  __shared__ double fk[kTabKnots];
  __shared__ double red[kBuildT / kWave][3];
  __shared__ int32_t scan[kBuildT];
  __shared__ uint16_t cell[kTabCells];
  __shared__ int sh_bad, sh_wide, sh_n, sh_max;
  const int q = q0 + (int)blockIdx.y, c = blockIdx.x;
  if (q >= cfirst[k]) return;
  const int4 ck = chunk[q];
  const int m = ck.z;
  const int tid = threadIdx.x;
  TabHead* hd = head + (size_t)blockIdx.y * d + c;
  if (tid == 0) sh_bad = sh_wide = 0;
  __syncthreads();
  int P = 1;
  while (P < m) P <<= 1;
  double wt = 0.0, wneg = 0.0, wother = 0.0;
  for (int r = tid; r < P; r += kBuildT) {
    float y = __builtin_inff(), wr = 0.0f;
    if (r < m) {
      y = Y32[(size_t)(ck.y + r) * DM + c];
      wr = w[ck.y + r];
      const float ay = fabsf(y);
      if (M == kManh ? !(ay <= kManhMax) : !(y == 0.0f || (ay >= kTabMin && ay <= kTabMax))) sh_bad = 1;
      if (!(wr <= kTabMax)) sh_bad = 1;
      if (!(ay <= kPairMax)) sh_wide = 1;
      wt += (double)wr;
      if (y < 0.0f) wneg += (double)wr;
      if (y != 0.0f) wother += (double)wr;
    }
    ys[r] = y == 0.0f ? 0.0f : y;  // (-0 to 0)
    ws[r] = wr;
  }
  wt = wave_sum_f64(wt);
  wneg = wave_sum_f64(wneg);
  wother = wave_sum_f64(wother);
  if ((tid & 63) == 0) {
    red[tid >> 6][0] = wt;
    red[tid >> 6][1] = wneg;
    red[tid >> 6][2] = wother;
  }
  __syncthreads();
  wt = wneg = wother = 0.0;
  for (int i = 0; i < kBuildT / kWave; ++i) {
    wt += red[i][0];
    wneg += red[i][1];
    wother += red[i][2];
  }
  if (sh_bad) {  // block-uniform
    if (tid == 0) hd->K = sh_wide ? -1 : 0;
    return;
  }
  // bitonic sort, ascending (padding +inf at the end)
  for (int size = 2; size <= P; size <<= 1)
    for (int st = size >> 1; st > 0; st >>= 1) {
      __syncthreads();
      for (int i = tid; i < P / 2; i += kBuildT) {
        const int a = 2 * i - (i & (st - 1)), b = a + st;
        const bool up = (a & size) == 0;
        const float ya = ys[a], yb = ys[b];
        if ((ya > yb) == up && ya != yb) {
          ys[a] = yb;
          ys[b] = ya;
          const float t = ws[a];
          ws[a] = ws[b];
          ws[b] = t;
        }
      }
    }
  __syncthreads();
  // exclusive scan of one count per thread; returns the thread's start, sh_n the total
  auto block_scan = [&](int v) {
    scan[tid] = v;
    __syncthreads();
    for (int o = 1; o < kBuildT; o <<= 1) {
      const int u = tid >= o ? scan[tid - o] : 0;
      __syncthreads();
      scan[tid] += u;
      __syncthreads();
    }
    const int excl = tid ? scan[tid - 1] : 0;
    if (tid == kBuildT - 1) sh_n = scan[kBuildT - 1];
    __syncthreads();
    return excl;
  };
  const int per = (m + kBuildT - 1) / kBuildT;
  const int r0 = tid * per < m ? tid * per : m, r1 = r0 + per < m ? r0 + per : m;
  const size_t base = tab_base(chunk, q, q0) * (size_t)d + (size_t)c * (size_t)(2 * m + kTabExtra);
  float* oy = tabY + base;
  double2* og = (double2*)tabG + base;

  uint16_t* ol = tabL + ((size_t)blockIdx.y * d + c) * kTabCells;
  // the lookup over the K knots kn: cell starts (byte offsets) to ol; the steps to L
  float inv = 0.0f, off = 0.0f;
  auto lookup = [&](int K) {
    const float z0 = kn[0];
    inv = (float)kTabCells / (kn[K - 1] - z0);
    off = -z0 * inv;
    if (tid == 0) sh_max = 0;
    for (int b = tid; b < kTabCells; b += kBuildT) cell[b] = 0;
    __syncthreads();
    for (int i = tid; i < K; i += kBuildT) {
      const int b0 = tab_cell(kn[i], inv, off), b1 = i + 1 < K ? tab_cell(kn[i + 1], inv, off) : kTabCells - 1;
      for (int b = b0 + 1; b <= b1; ++b) cell[b] = (uint16_t)i;
    }
    __syncthreads();
    int mx = 0;
    for (int b = tid; b < kTabCells; b += kBuildT) {
      const int hi = b + 1 < kTabCells ? (int)cell[b + 1] : K - 1;
      mx = hi - (int)cell[b] > mx ? hi - (int)cell[b] : mx;
    }
    atomicMax(&sh_max, mx);
    __syncthreads();
    for (int b = tid; b < kTabCells; b += kBuildT) ol[b] = (uint16_t)(4 * cell[b]);
    int L = 0;
    while ((1 << L) - 1 < sh_max) ++L;
    return L;
  };

  if constexpr (M == kManh) {
    int cntd = 0;
    for (int r = r0; r < r1; ++r) cntd += r == 0 || ys[r] != ys[r - 1];
    int at = block_scan(cntd);
    for (int r = r0; r < r1; ++r)
      if (r == 0 || ys[r] != ys[r - 1]) kn[at++] = ys[r];
    int K = sh_n;
    __syncthreads();
    if (K == 1) {  // one value: a second knot makes an interval
      if (tid == 0) kn[1] = kn[0] + fmaxf(1.0f, fabsf(kn[0]));
      K = 2;
      __syncthreads();
    }
    for (int i = tid; i < K; i += kBuildT) {
      const double t = (double)kn[i];
      double f = 0.0;
      for (int r = 0; r < m; ++r) f += (double)ws[r] * fabs(t - (double)ys[r]);
      fk[i] = f;
    }
    __syncthreads();
    for (int i = tid; i < K; i += kBuildT) {
      oy[i] = kn[i];
      if (i + 1 < K) {
        const double ig = 1.0 / ((double)kn[i + 1] - (double)kn[i]);
        og[i] = double2{fk[i] * ig, fk[i + 1] * ig};
      }
    }
    const int L = lookup(K);
    if (tid == 0) *hd = TabHead{K, L, inv, off, kn[0], kn[K - 1], (float)wt, 0.f};
  } else {
    // first index of the values >= 0 and > 0
    int nneg = 0, nzero = 0;
    {
      int lo = 0, hi = m;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (ys[mid] < 0.0f) lo = mid + 1; else hi = mid;
      }
      nneg = lo;
      hi = m;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (ys[mid] <= 0.0f) lo = mid + 1; else hi = mid;
      }
      nzero = lo - nneg;
    }
    const int p0 = nneg + nzero;  // positives: [p0, m)
    const double wpos = wother - wneg;
    const double Yp = p0 < m ? 2.0 * (double)ys[m - 1] : 1.0, Yn = nneg > 0 ? -2.0 * (double)ys[0] : 1.0;
    const double up = p0 < m ? (double)ys[p0] : 1.0, un = nneg > 0 ? -(double)ys[nneg - 1] : 1.0;
    // f at signed table position z
    auto f_at = [&](double z) {
      const bool neg = z < 0.0;
      const double Y = neg ? Yn : Yp;
      double t = fabs(z);
      if (t >= 2.0 * Y) return wt;   // |t| -> infinity
      if (t > Y) t = Y / (2.0 - t / Y);
      const int a = neg ? 0 : p0, b = neg ? nneg : m;
      double f = neg ? wt - wneg : wt - wpos;
      if (t == 0.0) return wt;  // the limit from either side
      // t as th + tl: th - y is exact for the y next to t, and tl matters there
      const float th = (float)t, tl = (float)(t - (double)th);
      int r = a;
      for (; r + 4 <= b; r += 4) {
        float s = 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float y = fabsf(ys[r + e]);
          s = fmaf(ws[r + e], canb_term(fabsf((th - y) + tl), th + y), s);
        }
        f += (double)s;
      }
      for (; r < b; ++r) {
        const float y = fabsf(ys[r]);
        f += (double)(ws[r] * canb_term(fabsf((th - y) + tl), th + y));
      }
      return f;
    };
    // base knots: -2 Yn, -Yn, the distinct negatives, 0, the distinct positives, Yp, 2 Yp
    int cntd = 0;
    for (int r = r0; r < r1; ++r) cntd += ys[r] != 0.0f && (r == 0 || ys[r] != ys[r - 1]);
    int at = block_scan(cntd);
    const int nd = sh_n;
    // of them negative: the distinct values before p0
    float* bk = kn + kTabMost;  // base knots wait at the end of kn
    if (tid == 0) {
      bk[0] = (float)(-2.0 * Yn);
      bk[1] = (float)-Yn;
      bk[nd + 3] = (float)Yp;
      bk[nd + 4] = (float)(2.0 * Yp);
    }
    for (int r = r0; r < r1; ++r)
      if (ys[r] != 0.0f && (r == 0 || ys[r] != ys[r - 1])) {
        bk[2 + at + (ys[r] > 0.0f ? 1 : 0)] = ys[r];
        if (ys[r] > 0.0f && (r == p0)) bk[2 + at] = 0.0f;  // 0 before the first positive
        ++at;
      }
    if (p0 == m && tid == 0) bk[2 + nd] = 0.0f;
    __syncthreads();
    const int nb = nd + 5;
    for (int i = tid; i < nb; i += kBuildT) fk[i] = f_at((double)bk[i]);
    __syncthreads();
    // parts of the segment from base knot i: its length in ln(t + u) over the step
    auto seg = [&](int i, double& a, double& u, double& len, bool& tail, bool& neg) {
      const double za = (double)bk[i], zb = (double)bk[i + 1];
      neg = zb <= 0.0;
      const double Y = neg ? Yn : Yp;
      u = neg ? un : up;
      const double lo = neg ? -zb : za, hi = neg ? -za : zb;
      tail = hi > Y;
      a = lo;
      len = tail ? 0.6931471805599453 : log((hi + u) / (lo + u));
      const bool none = neg ? nneg == 0 : p0 == m;
      if (none) return 1;
      const double fm = fmin(fk[i], fk[i + 1]) / wt;
      const double h = (double)kCanbStep * sqrt(sqrt(fmax(fm, (double)kCanbFloor)));
      const double ns = ceil(len / h);
      return ns < 4096.0 ? (int)ns : 4096;
    };
    const int pers = (nb - 1 + kBuildT - 1) / kBuildT;
    const int s0 = tid * pers < nb - 1 ? tid * pers : nb - 1, s1 = s0 + pers < nb - 1 ? s0 + pers : nb - 1;
    int tot = 0;
    double a, u, len;
    bool tail, neg;
    for (int i = s0; i < s1; ++i) tot += seg(i, a, u, len, tail, neg);
    int pos = block_scan(tot);
    const int K = sh_n + 1;
    const int room = 2 * m + kTabExtra;
    if (K >= room || K > kTabMost) {  // block-uniform
      if (tid == 0) hd->K = 0;
      return;
    }
    for (int i = s0; i < s1; ++i) {
      const int ns = seg(i, a, u, len, tail, neg);
      const double Y = neg ? Yn : Yp;
      kn[pos] = bk[i];
      for (int e = 1; e < ns; ++e) {
        // magnitude rises away from 0: on the negative side the parts run from
        // the far end
        const double x = (double)(neg ? ns - e : e) / (double)ns;
        const double mag = tail ? Y * (3.0 - 2.0 * exp(-len * x)) : (a + u) * exp(len * x) - u;
        kn[pos + e] = (float)(neg ? -mag : mag);
      }
      pos += ns;
    }
    if (tid == 0) kn[K - 1] = bk[nb - 1];
    __syncthreads();
    for (int i = tid; i < K; i += kBuildT) fk[i] = f_at((double)kn[i]);
    __syncthreads();
    bool bad = false;
    for (int i = tid; i < K; i += kBuildT) {
      oy[i] = kn[i];
      if (i + 1 < K) {
        const double z = (double)kn[i], gap = (double)kn[i + 1] - z;
        bad = bad || !(gap > 0.0);
        const double fa = fk[i], fb = fk[i + 1];
        const double r1v = f_at(z + 0.25 * gap) - (0.75 * fa + 0.25 * fb);
        const double r2v = f_at(z + 0.75 * gap) - (0.25 * fa + 0.75 * fb);
        double c1 = (r2v - r1v) * (32.0 / 3.0), c0 = r1v * (16.0 / 3.0) - 0.25 * c1;
        const double ig = 1.0 / gap;
        // Knots next to each other at small magnitudes: c1 ig^3 can pass the
        // float32 range.  The residual's own c1 is at most about Wt (gap /
        // 2^-30)^3, which Wt <= 2^30 keeps inside it, so such a c1 is the
        // rounding of f alone, and the mean of the two residuals serves.
        if (!(fabs(c1 * ig * ig * ig) <= (double)FLT_MAX)) {
          c1 = 0.0;
          c0 = (r1v + r2v) * (8.0 / 3.0);
        }
        og[i] = double2{fa * ig, fb * ig};
        tabC[base + i] = float2{(float)(c0 * ig * ig), (float)(c1 * ig * ig * ig)};
      }
    }
    if (bad) sh_bad = 1;  // two knots fell on one float
    float zero = 0.0f;
    if (tid == 0) {
      // f jumps at 0 where the sample has zeros: f(0) is the sum of the other
      // weights.  An element's 0 takes the record past the last interval,
      // E (f(0) / E), E a power of two above every z (the search stops there).
      const float E = __uint_as_float((__float_as_uint((float)(4.0 * Yp)) & 0x7f800000u) + 0x00800000u);
      if (nzero > 0) zero = E;
      og[K - 1] = double2{wother / (double)E, 0.0};
      tabC[base + K - 1] = float2{0.0f, 0.0f};
    }
    const int L = lookup(K);
    if (tid == 0)
      *hd = TabHead{sh_bad ? 0 : K, L, inv, off, -(float)Yn, (float)Yp, 0.f, zero};
  }
}

// ----------------------------------------------------------------------------
// XT[c][i] = coordinate c of the element at position i0 + i, i < R (row length
// R; position p is row perm[p] of X, null: row p).  In cluster order the
// elements of a wave lie near each other, so that many of its lanes read the
// same words of a table.
// ----------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_tab_transpose(const float* __restrict__ X,
                                                       const int32_t* __restrict__ perm, int64_t i0, int R, int d,
                                                       float* __restrict__ XT) {
  __shared__ float t[64][65];
  __shared__ int rows[64];
  const int r0 = blockIdx.x * 64, c0 = blockIdx.y * 64;
  const int nr = R - r0 < 64 ? R - r0 : 64, nc = d - c0 < 64 ? d - c0 : 64;
  if ((int)threadIdx.x < nr) {
    const int64_t p = i0 + r0 + threadIdx.x;
    rows[threadIdx.x] = perm != nullptr ? perm[p] : (int)p;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < nr * nc; q += 256) {
    const int r = q / nc, c = q - r * nc;
    t[r][c] = X[(size_t)rows[r] * d + c0 + c];
  }
  __syncthreads();
  for (int q = threadIdx.x; q < 64 * nc; q += 256) {
    const int c = q >> 6, r = q & 63;
    if (r < nr) XT[(size_t)(c0 + c) * R + r0 + r] = t[r][c];
  }
}

// ----------------------------------------------------------------------------
// n = 1e6, d = 32, k = 16, S = 4,764 Manhattan: Phase 2 5.53 -> 0.77 ms, of
// which this kernel 0.59 (8.6e11 table evaluations a second); n = 5e5, d = 64,
// k = 64, S = 9,337 Canberra 39.6 -> 3.36 ms, this kernel 2.82, the tables 0.30.
// Float32 records and sums would save a fifth and a seventh of it, but have 1.5
// times the direct sums' error at d <= 24, t = 500.  With them, where this form
// took 0.52 and 2.51 ms: searching in halves alone 0.85 / 3.59, 512 threads a
// block 0.61 / 2.95, 1024 threads 0.60 / 4.31, 16 elements a thread 0.77 / 3.89.
//
// One block per (tile of kEvalT E elements, cluster): for each of the
// cluster's chunks in the group, and each coordinate, the table into LDS and
// the tile's elements through it.  Wd [k][R]: assigned by the cluster's first
// chunk (or where it has none), added to by the others.
// ----------------------------------------------------------------------------
// Canberra's eight elements a thread hold 92 vector registers, five waves per
// SIMD (the direct sums below would take 99: four waves, 3.92 -> 4.29 ms).  One
// and two elements a thread would fill the SIMD's eight, and there the scalar
// registers count: a wave holds 16 more than the kernel names, so 96 let seven
// run (n = 55,822, d = 77, k = 44, t = 84: 106 490 us, 100 444, 96 385; forced to
// eight waves many spill, n = 68,362, d = 135, k = 17, t = 61 414 -> 525, 96 382).
template <int M, int E>
constexpr int kEvalWaves = M == kCanb && E == 8 ? 5 : 1;
constexpr int kEvalSgprs = 96;
static_assert(kEvalT == kTabCells / 2, "k_tab_eval: a word of cell starts a thread");
static_assert(kTabPad == kWave, "k_tab_eval: a wave writes the padding");

template <int M, int E>
__global__ __launch_bounds__(kEvalT) __attribute__((amdgpu_waves_per_eu(kEvalWaves<M, E>), amdgpu_num_sgpr(kEvalSgprs))) void k_tab_eval(const float* __restrict__ XT, int R, int d,
                                                     const int4* __restrict__ chunk,
                                                     const int32_t* __restrict__ cfirst, int k, int q0, int q1,
                                                     const TabHead* __restrict__ head,
                                                     const float* __restrict__ tabY, const double* __restrict__ tabG,
                                                     const float2* __restrict__ tabC,
                                                     const uint16_t* __restrict__ tabL,
                                                     const float* __restrict__ Y32, int DM,
                                                     const float* __restrict__ w, int tiles, int knots,
                                                     double* __restrict__ Wd) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  // knots (and kTabPad times +inf, so that steps past the end find nothing),
  // cell starts, records
  float* ly = (float*)lds;
  uint16_t* lc = (uint16_t*)(lds + (size_t)(knots + kTabPad) * 4);
  unsigned char* lg = lds + (size_t)(knots + kTabPad) * 4 + kTabCells * 2;  // g, h
  unsigned char* lp = lg + (size_t)knots * 16;                                // Canberra: c0, c1
  // eight XCDs take the blocks in turn: the blocks of one tile (its k
  // clusters) go to one XCD, whose L2 then holds the tile's columns
  const int b = blockIdx.x, grp = b / (8 * k), in = b - grp * 8 * k;
  const int tile = grp * 8 + (in & 7), j = in >> 3;
  if (tile >= tiles) return;
  const int last = cfirst[k];
  int ca = cfirst[j], cb = cfirst[j + 1];
  const bool assign = ca >= q0 || q0 == 0;  // nothing of this cluster was summed before this group
  const bool mine = q0 == 0 ? true : (ca < q1 && cb > q0);
  ca = ca > q0 ? ca : q0;
  cb = cb < q1 ? cb : q1;
  cb = cb < last ? cb : last;
  if (!mine) return;
  const int e0 = tile * (kEvalT * E) + threadIdx.x;
  double acc[E];
#pragma unroll
  for (int e = 0; e < E; ++e) acc[e] = 0.0;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  int refused = 0;
  for (int q = ca; q < cb; ++q) {
    const int4 ck = chunk[q];
    const int m = ck.z;
    const size_t base = tab_base(chunk, q, q0) * (size_t)d;
    for (int c = 0; c < d; ++c) {
      const TabHead hd = head[(size_t)(q - q0) * d + c];
      float x[E];
      const float* xc = XT + (size_t)c * R;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int i = e0 + e * kEvalT;
        x[e] = xc[i < R ? i : R - 1];
      }
      const int K = hd.K;
      if (K <= 0) {  // block-uniform
        refused = 1;
        continue;
      }
      __syncthreads();
      {
        const size_t tb = base + (size_t)c * (size_t)(2 * m + kTabExtra);
        for (int i = threadIdx.x; i < K; i += kEvalT) {
          ly[i] = tabY[tb + i];
          ((double2*)lg)[i] = ((const double2*)tabG)[tb + i];
          if (M == kCanb) ((float2*)lp)[i] = tabC[tb + i];
        }
        if (wave == 0) {
          ly[K + threadIdx.x] = __builtin_inff();
          if (M == kCanb && __float_as_int(hd.zero) != 0) ly[K] = hd.zero;  // (after the wave's own +inf)
        }
        ((uint32_t*)lc)[threadIdx.x] = ((const uint32_t*)(tabL + ((size_t)(q - q0) * d + c) * kTabCells))[threadIdx.x];
      }
      __syncthreads();
      bool odd = false;  // Canberra: a value past 2^62 or not finite
      if (M == kCanb) {
#pragma unroll
        for (int e = 0; e < E; ++e) odd = odd || !(fabsf(x[e]) <= 0x1p62f);
        odd = __any(odd);
      }
      if (!odd) {
        float z[E];
        bool far = false;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          if (M == kManh) {
            z[e] = __builtin_amdgcn_fmed3f(x[e], hd.lo, hd.hi);
          } else {
            z[e] = x[e];
            far = far || x[e] > hd.hi || x[e] < hd.lo;
          }
        }
        if (M == kCanb && __any(far)) {
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const float ax = fabsf(x[e]), Y = x[e] < 0.0f ? -hd.lo : hd.hi;
            const float zt = fmaf(-Y, canb_term(Y, ax), 2.0f * Y);  // Y (2 - Y / |x|)
            z[e] = ax > Y ? copysignf(fminf(zt, 2.0f * Y), x[e]) : x[e];
          }
        }
        // byte offset of the interval's first knot: the last knot at or below
        // z among knots 0 .. K - 2 (knot 0 is below every z)
        int at[E];
        if (hd.L <= kTabSteps) {
#pragma unroll
          for (int e = 0; e < E; ++e) at[e] = (int)lc[tab_cell(z[e], hd.inv, hd.off)];
#pragma unroll
          for (int l = kTabSteps - 1; l >= 0; --l) {
            if (l < hd.L) {  // uniform
#pragma unroll
              for (int e = 0; e < E; ++e) {
                const float y = *(const float*)((const unsigned char*)ly + at[e] + (4 << l));
                at[e] += y <= z[e] ? (4 << l) : 0;
              }
            }
          }
#pragma unroll
          for (int e = 0; e < E; ++e) at[e] = at[e] < 4 * (K - 2) ? at[e] : 4 * (K - 2);
        } else {
#pragma unroll
          for (int e = 0; e < E; ++e) at[e] = 0;
          for (int len = K - 1; len > 1;) {
            const int half = len >> 1;
#pragma unroll
            for (int e = 0; e < E; ++e) {
              const int mid = at[e] + 4 * half;
              at[e] = *(const float*)((const unsigned char*)ly + mid) <= z[e] ? mid : at[e];
            }
            len -= half;
          }
        }
        if (M == kCanb && __float_as_int(hd.zero) != 0) {  // uniform
#pragma unroll
          for (int e = 0; e < E; ++e) at[e] = x[e] == 0.0f ? 4 * (K - 1) : at[e];
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const float* yp = (const float*)((const unsigned char*)ly + at[e]);
          const float ya = yp[0], yb = yp[1];
          const double2 g = *(const double2*)(lg + 4 * at[e]);
          const double zd = (double)z[e];
          acc[e] = fma((double)yb - zd, g.x, acc[e]);
          acc[e] = fma(zd - (double)ya, g.y, acc[e]);
          if constexpr (M == kCanb) {
            const float2 p = *(const float2*)(lp + 2 * at[e]);
            const float a = yb - z[e], bb = z[e] - ya;
            acc[e] += (double)(a * bb * fmaf(p.y, bb, p.x));
          }
        }
        if (M == kManh) {
          bool out = false;
#pragma unroll
          for (int e = 0; e < E; ++e) out = out || x[e] != z[e];
          if (__any(out)) {
#pragma unroll
            for (int e = 0; e < E; ++e) acc[e] = fma((double)hd.Wt, fabs((double)x[e] - (double)z[e]), acc[e]);
          }
        }
      } else {
        // Canberra, a wave with an element past the table's map: as above, from
        // memory
        const float* yc = Y32 + (size_t)ck.y * DM + c;
        const float* wc = w + ck.y;
        for (int g0 = 0; g0 < m; g0 += 32) {
          const int g1 = g0 + 32 < m ? g0 + 32 : m;
          float s[E];
#pragma unroll
          for (int e = 0; e < E; ++e) s[e] = 0.0f;
          for (int r = g0; r < g1; ++r) {
            const float y = yc[(size_t)r * DM], wr = wc[r];
#pragma unroll
            for (int e = 0; e < E; ++e) {
              const float den = fmaxf(fabsf(x[e]) + fabsf(y), FLT_MIN);
              s[e] = fmaf(wr, fabsf(x[e] - y) * __builtin_amdgcn_rcpf(den), s[e]);
            }
          }
#pragma unroll
          for (int e = 0; e < E; ++e) acc[e] += (double)s[e];
        }
      }
    }
  }
  // the refused tables, after all others (a loop of its own holds fewer scalar
  // registers than one within the chunks' loop)
  for (int q = refused != 0 ? ca : cb; q < cb; ++q) {
    const int4 ck = chunk[q];
    const int m = ck.z;
    for (int c = 0; c < d; ++c) {
      const int K = head[(size_t)(q - q0) * d + c].K;
      if (K > 0) continue;
      // the values and weights in pairs of rows
      __syncthreads();
      for (int i = threadIdx.x; i < ((m + 1) & ~1); i += kEvalT)
        ((float2*)lds)[i] = i < m ? float2{Y32[(size_t)(ck.y + i) * DM + c], w[ck.y + i]} : float2{1.0f, 0.0f};
      float x[E];
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int i = e0 + e * kEvalT;
        x[e] = XT[(size_t)c * R + (i < R ? i : R - 1)];
      }
      __syncthreads();
      // directly, 32 rows in float32, then float64.  Canberra: two rows with
      // one reciprocal, (w0 n0 d1 + w1 n1 d0) / (d0 d1), where the wave's
      // elements and the values lie in what two factors allow (k_p2_valu pairs
      // coordinates the same way).  n = 200,000, d = 32, k = 16, t = 256, every
      // table refused: Canberra 8.95 -> 4.19 ms (pairs of coordinates by k_p2_valu 5.89)
      bool pairs = M == kCanb && K == 0;
      if (pairs) {
#pragma unroll
        for (int e = 0; e < E; ++e) pairs = pairs && fabsf(x[e]) >= 0x1p-62f && fabsf(x[e]) <= kPairMax;
        pairs = __all(pairs);
      }
      for (int g0 = 0; g0 < m; g0 += 32) {
        const int g1 = g0 + 32 < m ? g0 + 32 : m;
        float s[E];
#pragma unroll
        for (int e = 0; e < E; ++e) s[e] = 0.0f;
        const float4* yw = (const float4*)lds + g0 / 2;
        const int np = (g1 - g0 + 1) / 2;
        if (M == kManh) {
          for (int r = 0; r < np; ++r) {
            const float4 v = yw[r];
#pragma unroll
            for (int e = 0; e < E; ++e) {
              s[e] = fmaf(v.y, fabsf(x[e] - v.x), s[e]);
              s[e] = v.w != 0.0f ? fmaf(v.w, fabsf(x[e] - v.z), s[e]) : s[e];
            }
          }
        } else if (pairs) {
#pragma unroll 1
          for (int r = 0; r < np; ++r) {
            const float4 v = yw[r];
#pragma unroll
            for (int e = 0; e < E; ++e) {
              const float d0 = fabsf(x[e]) + fabsf(v.x), d1 = fabsf(x[e]) + fabsf(v.z);
              const float n0 = v.y * fabsf(x[e] - v.x), n1 = v.w * fabsf(x[e] - v.z);
              s[e] = fmaf(fmaf(n0, d1, n1 * d0), __builtin_amdgcn_rcpf(d0 * d1), s[e]);
            }
          }
        } else {
          for (int r = g0; r < g1; ++r) {
            const float2 v = ((const float2*)lds)[r];
#pragma unroll
            for (int e = 0; e < E; ++e) {
              const float den = fmaxf(fabsf(x[e]) + fabsf(v.x), FLT_MIN);
              s[e] = fmaf(v.y, fabsf(x[e] - v.x) * __builtin_amdgcn_rcpf(den), s[e]);
            }
          }
        }
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] += (double)s[e];
      }
    }
  }
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = e0 + e * kEvalT;
    if (i < R) {
      double* o = Wd + (size_t)j * R + i;
      *o = assign ? acc[e] : *o + acc[e];
    }
  }
}

// ----------------------------------------------------------------------------
// a_hat, b_hat, s_hat of the elements at positions i0 .. i0 + R - 1 from their
// sums Wd [k][R]; a float64 partial of the sum of s_hat per kTabScore positions
// ----------------------------------------------------------------------------
__global__ __launch_bounds__(kTabScore) void k_tab_scores(const double* __restrict__ Wd, int64_t i0, int R,
                                                          const int32_t* __restrict__ perm,
                                                          const int32_t* __restrict__ labels,
                                                          const int32_t* __restrict__ csize, int k,
                                                          float* __restrict__ a_out, float* __restrict__ b_out,
                                                          float* __restrict__ s_out, float* __restrict__ What,
                                                          double* __restrict__ bpart) {
  __shared__ double sh[kTabScore / kWave];
  const int i = blockIdx.x * kTabScore + threadIdx.x;
  const bool valid = i < R;
  const int ir = valid ? i : R - 1;
  const int64_t e = perm != nullptr ? (int64_t)perm[i0 + ir] : i0 + ir;
  int own = labels[e];
  own = (unsigned)own < (unsigned)k ? own : 0;  // labels are checked before; stay in bounds
  double w_own = 0.0, bmin = __builtin_inf();
  for (int j = 0; j < k; ++j) {
    const double W = Wd[(size_t)j * R + ir];
    if (What != nullptr && valid) What[(size_t)e * k + j] = (float)W;
    const int sz = csize[j];
    if (j == own) {
      w_own = W;
    } else if (sz > 0) {
      const double bj = W / (double)sz;
      bmin = bj < bmin ? bj : bmin;
    }
  }
  const int szo = csize[own];
  const double a = szo > 1 ? w_own / (double)(szo - 1) : 0.0;
  const double mx = a > bmin ? a : bmin;
  const double s = (szo > 1 && mx > 0.0) ? (bmin - a) / mx : 0.0;
  if (valid) {
    if (a_out) a_out[e] = (float)a;
    if (b_out) b_out[e] = (float)bmin;
    if (s_out) s_out[e] = (float)s;
  }
  const double tot = block_sum_f64<kTabScore>(valid ? s : 0.0, sh);
  if (threadIdx.x == 0) bpart[i0 / kTabScore + blockIdx.x] = tot;
}

// ----------------------------------------------------------------------------
// Tables pay where the elements are many enough to share their construction
// and the clusters have more rows than an evaluation costs.  silh_scores,
// direct sums -> tables: n = 1,024, d = 8, k = 4, t = 64 Manhattan 100 -> 70 us,
// Canberra 131 -> 90; n = 262,144, d = 32, k = 64, t = 24 724 -> 533, 2203 ->
// 732; n = 1e6, d = 8, k = 16, t = 32 287 -> 243, 718 -> 285; n = 65,536, d = 32,
// k = 16, t = 64 472 -> 125, 985 -> 183.  Two or three clusters, or Canberra's
// tables of 512 and more rows at small n, take longer by tables (requests:
// Manhattan n = 1,024, d = 64, k = 2, t = 16 175 -> 256, n = 100,000, d = 64, k = 2,
// t = 16 208 -> 292; Canberra n = 2,048, d = 4, k = 2, t = 1,024 646 -> 709, n = 51,543,
// d = 26, k = 3, t = 21 241 -> 279), but they add in float64 where the direct sums
// do in float32: 8.4e-8 -> 3.5e-8, 1.0e-7 -> 5.9e-8, 8.5e-7 -> 1.6e-7 off 64 bits
// at such sizes.  Fewer elements or rows are summed directly, also where many
// clusters would make the tables faster (Manhattan n = 841, d = 108, k = 12, t = 70
// 1,960 -> 299).
bool tab_pays(int metric, int64_t n, int k, int64_t t) {
  if (metric != kManh && metric != kCanb) return false;
  const int64_t per = n / k, m = t < per ? t : per;
  return n >= 1024 && m >= 16;
}

size_t tab_bytes(const TabPlan& p, int k, int d) {
  return (size_t)p.chunks * 16 + ((size_t)k + 1) * 4 + (size_t)p.group * d * (sizeof(TabHead) + 2 * kTabCells) +
         p.knots * (size_t)(1 + p.rw) * 4 + (size_t)p.rows * ((size_t)d * 4 + (size_t)k * 8) + 2048;
}

TabPlan tab_plan(int metric, int64_t n, int d, int k, int64_t S_pad, int64_t max_rows, bool pieces) {
  TabPlan p;
  const int RW = metric == kManh ? 4 : 6;  // floats per record: g, h (float64), Canberra c0, c1
  const size_t kb = (size_t)(1 + RW) * sizeof(float);
  p.chunks = ceil_div(S_pad, kTabRows) + k;
  const int64_t mr = max_rows < kTabRows ? max_rows : kTabRows;
  // one chunk's tables at most (and a cluster's padding rows between chunks)
  const size_t chunk_knots = (size_t)(2 * mr + kTabExtra + 2 * kSamplePad);
  const size_t per = chunk_knots * d * kb;
  int64_t g = (int64_t)(kTabGroupBytes / per);
  g = g < 1 ? 1 : g;
  p.group = g < p.chunks ? g : p.chunks;
  size_t knots = (size_t)p.group * chunk_knots;
  const size_t all = (size_t)(2 * S_pad + kTabExtra * p.chunks);
  knots = knots < all ? knots : all;
  p.knots = knots * (size_t)d;
  int64_t R = kTabWork / (k > 2 * d ? k : 2 * d);  // sums and twice the transposed floats
  p.wait = pieces;
  if (pieces) {
    const int64_t r = kPieceEvals / ((p.chunks > k ? p.chunks - k + ceil_div(k, 2) : k) * d);
    R = r < R ? r : R;
  }
  R = R / (8 * kEvalT) * (8 * kEvalT);
  R = R < kTabScore ? kTabScore : R;
  p.rows = R < n ? R : n;
  p.rw = RW;
  // the longest table: LDS of the evaluation (Manhattan has no refinement)
  p.max_knots = (int)(metric == kManh ? mr + 2 : 2 * mr + kTabExtra < kTabMost + 1 ? 2 * mr + kTabExtra : kTabMost + 1);
  p.max_knots = (p.max_knots + 3) & ~3;  // (the records after it are 16-byte aligned)
  return p;
}

template <int M, int E>
static void launch_eval(hipStream_t st, const TabBufs& B, const TabPlan& p, int R, int d, int k, int q0, int q1,
                        const float* Y32, int DM, const float* w) {
  const int tiles = (int)ceil_div(R, kEvalT * E);
  const int grid = (int)ceil_div(tiles, 8) * 8 * k;
  const size_t lds = (size_t)p.max_knots * (size_t)(1 + p.rw) * sizeof(float) + 4 * kTabPad + 2 * kTabCells;
  hipLaunchKernelGGL((k_tab_eval<M, E>), dim3((unsigned)grid), dim3(kEvalT), lds, st, B.XT, R, d, (const int4*)B.chunk,
                     B.cfirst, k, q0, q1, (const TabHead*)B.head, B.Y, B.G, (const float2*)B.C, B.L, Y32, DM, w, tiles, p.max_knots, B.Wd);
}

template <int M>
static void launch_tab(hipStream_t st, int DM, const P2Args& A, const TabPlan& p, const TabBufs& B) {
  const int n = A.n, d = A.d, k = A.k;
  hipLaunchKernelGGL(k_tab_chunks, dim3(1), dim3(1024), 0, st, A.sp_off, A.cnt, k, (int)p.chunks, (int4*)B.chunk,
                     B.cfirst);
  for (int64_t i0 = 0; i0 < n; i0 += p.rows) {
    const int R = n - i0 < p.rows ? (int)(n - i0) : (int)p.rows;
    hipLaunchKernelGGL(k_tab_transpose, dim3((unsigned)ceil_div(R, 64), (unsigned)ceil_div(d, 64)), dim3(256), 0, st,
                       A.X, A.perm, i0, R, d, B.XT);
    for (int64_t q0 = 0; q0 < p.chunks; q0 += p.group) {
      const int64_t nq = p.chunks - q0 < p.group ? p.chunks - q0 : p.group;
      if (i0 == 0 || p.group < p.chunks)
        hipLaunchKernelGGL(k_tab_build<M>, dim3((unsigned)d, (unsigned)nq), dim3(kBuildT), 0, st, A.Y, DM, d, A.w,
                           (const int4*)B.chunk, B.cfirst, k, (int)q0, (TabHead*)B.head, B.Y, B.G, (float2*)B.C, B.L);
      // elements per thread: as many as leave eight blocks per CU
      if ((int64_t)R * k >= (int64_t)2048 * kEvalT * 8)
        launch_eval<M, M == kManh ? 4 : 8>(st, B, p, R, d, k, (int)q0, (int)(q0 + nq), A.Y, DM, A.w);
      else if ((int64_t)R * k >= (int64_t)2048 * kEvalT * 2)
        launch_eval<M, 2>(st, B, p, R, d, k, (int)q0, (int)(q0 + nq), A.Y, DM, A.w);
      else
        launch_eval<M, 1>(st, B, p, R, d, k, (int)q0, (int)(q0 + nq), A.Y, DM, A.w);
    }
    hipLaunchKernelGGL(k_tab_scores, dim3((unsigned)ceil_div(R, kTabScore)), dim3(kTabScore), 0, st, B.Wd, i0, R,
                       A.perm, A.labels, A.csize, k, A.a, A.b, A.s, A.What, A.bpart);
    if (p.wait && i0 + p.rows < n && hipStreamSynchronize(st) != hipSuccess) return;
  }
}

size_t tab_head_bytes() { return sizeof(TabHead); }
size_t tab_cells() { return kTabCells; }

bool launch_phase2_tab(hipStream_t st, int metric, int DM, const P2Args& A, const TabPlan& p, const TabBufs& B) {
  if (A.n <= 0) return true;
  if (metric == kManh)
    launch_tab<kManh>(st, DM, A, p, B);
  else
    launch_tab<kCanb>(st, DM, A, p, B);
  return true;
}

}  // namespace silh
