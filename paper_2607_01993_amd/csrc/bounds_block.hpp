// The bounds of a block of elements (k_phase2_bounds.hip has the derivation), for
// the launch that writes the masks and for the probe that rides on the packing
// of the operands.
#pragma once
#include "device_common.hpp"
#include "silh_internal.hpp"

namespace silh {

constexpr int kBoundRec = 8;  // floats: Wt/|C| (-1: empty cluster), V, slack, E of D, E const, padding; then m_j [DM]

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

// Elements row0 .. row0 + 63 (in perm order), NW waves.  out: the masks of all
// groups; PROBE: one word, the number of clusters that the block's groups need.
// stop() is asked once, beside the first loads.
template <int DM, int NW, bool PROBE, class F>
__device__ __forceinline__ void bounds_block(const float* __restrict__ X, int n, int d,
                                             const int32_t* __restrict__ labels, const int32_t* __restrict__ perm,
                                             const float* __restrict__ rec, int k, int row0,
                                             uint32_t* __restrict__ out, F stop) {
  constexpr int NT = 64 * NW, LD = DM + 4;
  __shared__ __attribute__((aligned(16))) float xs[64 * LD];
  __shared__ float low[kBndKeep<DM>][64];
  __shared__ float um[NW][64];
  __shared__ uint32_t bits[2][128];  // k <= 4096
  __shared__ int rows[64];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int kw = (k + 31) >> 5;
  const int i = row0 + lane < n ? row0 + lane : n - 1;
  const int row = perm != nullptr ? perm[i] : i;
  if (stop()) return;
  if (wave == 0) rows[lane] = row;
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
  int own = labels[row];
  own = (unsigned)own < (unsigned)k ? own : 0;  // labels are checked before; stay in bounds
  __syncthreads();
  const float* xl = xs + lane * LD;
  constexpr size_t RS = (size_t)kBoundRec + DM;
  // |x - m_j|^2 of two clusters
  auto dist2 = [&](int j, int j2, float (&out)[2]) {
    const float* m0 = rec + (size_t)j * RS + kBoundRec;
    const float* m1 = rec + (size_t)j2 * RS + kBoundRec;
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
  if constexpr (PROBE) {
    if (wave == 0) {
      int c = 0;
      for (int q = lane; q < 2 * kw; q += kWave) {
        const int g = q / kw;
        if (row0 + 32 * g < n) c += __builtin_popcount(bits[g][q - g * kw]);
      }
      c = wave_sum_i32(c);
      if (lane == 0) *out = (uint32_t)c;
    }
    return;
  }
  for (int q = threadIdx.x; q < 2 * kw; q += NT) {
    const int g = q / kw, wd = q - g * kw;
    if (row0 + 32 * g < n) out[(size_t)(row0 / 32 + g) * kw + wd] = bits[g][wd];
  }
}

}  // namespace silh
