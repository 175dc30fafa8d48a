// One row of causal attention by one wave on the vector ALU: what the vector kernels do for every row, and what the
// matrix-core kernels fall back on for a row whose result is not finite.
//
// A matrix-core tile multiplies every key of the tile with every row of it and gives the keys behind the diagonal the
// weight 0.  That is the same sum as long as those keys and values are finite; an infinity or NaN among them turns the
// rows before it into NaN (0 x inf).  A row that really has a non-finite result is recomputed as well: the terms in which
// the matrix cores take a weight (attention_mfma.hip) do not add up to an infinity.  Either way the row becomes what
// these functions make of it, which never touch a key behind it.
#pragma once

#include <math.h>

#include "po_common.h"

namespace po {

// Row i of head `head`: o_row[dh] and *lse.  query(e) is element e of the row's query, scaled; SLOTS * 64 >= dh.
// All 64 lanes of the wave call it with the same arguments.
template <typename T, int SLOTS, typename Query>
__device__ __forceinline__ void attention_forward_row(Query query, const T* __restrict__ kbase, const T* __restrict__ vbase,
                                                      int ld, int i, int dh, int lane, T* __restrict__ o_row,
                                                      float* __restrict__ lse) {
  float m = -INFINITY, l = 0.f;
  float acc[SLOTS];
#pragma unroll
  for (int r = 0; r < SLOTS; ++r) acc[r] = 0.f;
  for (int j0 = 0; j0 <= i; j0 += kWave) {
    int j = j0 + lane;
    float sc = -INFINITY;
    if (j <= i) {
      const T* kr = kbase + (size_t)j * ld;
      float d = 0.f;
      for (int e = 0; e < dh; ++e) d = fmaf(query(e), to_f32(kr[e]), d);
      sc = d;
    }
    float mnew = fmaxf(m, wave_max(sc));
    float p = (j <= i) ? __expf(sc - mnew) : 0.f;
    float alpha = __expf(m - mnew);
    l = l * alpha + wave_sum(p);
#pragma unroll
    for (int r = 0; r < SLOTS; ++r) acc[r] *= alpha;
    int nj = min(kWave, i - j0 + 1);
    for (int jj = 0; jj < nj; ++jj) {
      float pj = __shfl(p, jj, kWave);
      const T* vr = vbase + (size_t)(j0 + jj) * ld;
#pragma unroll
      for (int r = 0; r < SLOTS; ++r) {
        int e = lane + kWave * r;
        if (e < dh) acc[r] = fmaf(pj, to_f32(vr[e]), acc[r]);
      }
    }
    m = mnew;
  }
  float inv = 1.0f / l;
#pragma unroll
  for (int r = 0; r < SLOTS; ++r) {
    int e = lane + kWave * r;
    if (e < dh) o_row[e] = from_f32<T>(acc[r] * inv);
  }
  if (lane == 0) *lse = m + __logf(l);
}

// Row i of dQ: dq_row[dh].  query(e) as above, upstream(e) element e of the row's dO.
template <typename T, int SLOTS, typename Query, typename Upstream>
__device__ __forceinline__ void attention_dq_row(Query query, Upstream upstream, const T* __restrict__ kbase,
                                                 const T* __restrict__ vbase, int ld, float lse_i, float delta_i, int i,
                                                 int dh, int lane, float scale, T* __restrict__ dq_row) {
  float acc[SLOTS];
#pragma unroll
  for (int r = 0; r < SLOTS; ++r) acc[r] = 0.f;
  for (int j0 = 0; j0 <= i; j0 += kWave) {
    int j = j0 + lane;
    float ds = 0.f;
    if (j <= i) {
      const T* kr = kbase + (size_t)j * ld;
      const T* vr = vbase + (size_t)j * ld;
      float sc = 0.f, dp = 0.f;
      for (int e = 0; e < dh; ++e) {
        sc = fmaf(query(e), to_f32(kr[e]), sc);
        dp = fmaf(upstream(e), to_f32(vr[e]), dp);
      }
      ds = __expf(sc - lse_i) * (dp - delta_i);
    }
    int nj = min(kWave, i - j0 + 1);
    for (int jj = 0; jj < nj; ++jj) {
      float dsj = __shfl(ds, jj, kWave);
      const T* kr = kbase + (size_t)(j0 + jj) * ld;
#pragma unroll
      for (int r = 0; r < SLOTS; ++r) {
        int e = lane + kWave * r;
        if (e < dh) acc[r] = fmaf(dsj, to_f32(kr[e]), acc[r]);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < SLOTS; ++r) {
    int e = lane + kWave * r;
    if (e < dh) dq_row[e] = from_f32<T>(acc[r] * scale);
  }
}

// ---- for the matrix-core kernels, whose waves own 32 rows with lane L holding part of row L % 32 -------------------
// The rows of which some lane says `bad`, one bit each, those from `rows` on left out.
__device__ __forceinline__ uint32_t rows_to_redo(bool bad, int rows) {
  const uint64_t b = __builtin_amdgcn_ballot_w64(bad);
  uint32_t m = __builtin_amdgcn_readfirstlane((uint32_t)b | (uint32_t)(b >> 32));
  return rows >= 32 ? m : rows <= 0 ? 0u : m & ((1u << rows) - 1u);
}

// Rows row0 + r for every set bit r of `redo`, with all operands in memory.
template <typename T, int DH>
__device__ __forceinline__ void redo_forward_rows(uint32_t redo, int row0, const T* __restrict__ qkv, T* __restrict__ o,
                                                  float* __restrict__ lse, int s, int h, int hkv, int group, int head,
                                                  float scale) {
  while (redo) {
    const int i = row0 + __builtin_ctz(redo), ld = h + 2 * hkv;
    redo &= redo - 1;
    int dh = DH, lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+s"(dh));  // a loop, not DH times its body
    const T* q = qkv + (size_t)i * ld + head * dh;
    const T* k = qkv + h + (head / group) * dh;
    attention_forward_row<T, (DH + kWave - 1) / kWave>([&](int e) { return to_f32(q[e]) * scale; }, k, k + hkv, ld, i, dh,
                                                       lane, o + (size_t)i * h + head * dh, lse + (size_t)head * s + i);
  }
}
template <typename T, int DH>
__device__ __forceinline__ void redo_dq_rows(uint32_t redo, int row0, const T* __restrict__ qkv, const T* __restrict__ d_o,
                                             const float* __restrict__ lse, const float* __restrict__ delta,
                                             T* __restrict__ dqkv, int s, int h, int hkv, int group, int head, float scale) {
  while (redo) {
    const int i = row0 + __builtin_ctz(redo), ld = h + 2 * hkv;
    redo &= redo - 1;
    int dh = DH, lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+s"(dh));
    const T* q = qkv + (size_t)i * ld + head * dh;
    const T* g = d_o + (size_t)i * h + head * dh;
    const T* k = qkv + h + (head / group) * dh;
    attention_dq_row<T, (DH + kWave - 1) / kWave>([&](int e) { return to_f32(q[e]) * scale; },
                                                  [&](int e) { return to_f32(g[e]); }, k, k + hkv, ld,
                                                  lse[(size_t)head * s + i], delta[(size_t)head * s + i], i, dh, lane, scale,
                                                  dqkv + (size_t)i * ld + head * dh);
  }
}

}  // namespace po
