// Linear interpolation of the LS pair estimates ([l(2)][u][n][b] per slot) to one RE: between the pair centres
// 4 n + 1 + delta in frequency (flat beyond the outermost), between the two DMRS symbols in time (flat outside).
#pragma once
#include "common.h"

namespace {

struct LsPoint {
  int n0, n1;        // pairs on either side of the subcarrier
  float w;           // weight of n1
  float wt0, wt1;    // weights of the two DMRS symbols
};

__device__ __forceinline__ LsPoint ls_point(int s, int t, int delta, int np) {
  LsPoint q;
  const int p0 = 1 + delta, plast = 4 * (np - 1) + 1 + delta;
  if (s <= p0) { q.n0 = 0; q.w = 0.f; }
  else if (s >= plast) { q.n0 = np - 1; q.w = 0.f; }
  else { q.n0 = (s - 1 - delta) / 4; q.w = (float)(s - (4 * q.n0 + 1 + delta)) * 0.25f; }
  q.n1 = q.n0 + 1 < np ? q.n0 + 1 : q.n0;
  if (t <= NRX_DMRS0) { q.wt0 = 1.f; q.wt1 = 0.f; }
  else if (t >= NRX_DMRS1) { q.wt0 = 0.f; q.wt1 = 1.f; }
  else { q.wt0 = (float)(NRX_DMRS1 - t) / 9.f; q.wt1 = (float)(t - NRX_DMRS0) / 9.f; }
  return q;
}

// (fused products spelled out: every user of the estimate gets the same bits)
__device__ __forceinline__ float2 ls_mix_freq(const LsPoint &q, float2 a0, float2 a1) {
  return make_float2(fmaf(1.f - q.w, a0.x, q.w * a1.x), fmaf(1.f - q.w, a0.y, q.w * a1.y));
}
__device__ __forceinline__ float2 ls_mix_time(const LsPoint &q, float2 h0, float2 h1) {
  return make_float2(fmaf(q.wt0, h0.x, q.wt1 * h1.x), fmaf(q.wt0, h0.y, q.wt1 * h1.y));
}

// estimate of UE u at antenna b from the slot's pairs P
__device__ __forceinline__ float2 ls_interp(const float2 *P, const LsPoint &q, int U, int u, int B, int b, int np) {
  float2 hl[2];
#pragma unroll
  for (int li = 0; li < 2; ++li) {
    const float2 *r = P + ((int64_t)li * U + u) * np * B + b;
    hl[li] = ls_mix_freq(q, r[(int64_t)q.n0 * B], r[(int64_t)q.n1 * B]);
  }
  return ls_mix_time(q, hl[0], hl[1]);
}

}  // namespace
