// One row of causal attention by one wave on the vector ALU: what the vector kernels do for every row, and what the
// matrix-core kernels fall back on for a row whose result is not finite.
//
// A matrix-core tile multiplies every key of the tile with every row of it and gives the keys behind the diagonal the
// weight 0.  That is the same sum as long as those keys and values are finite; an infinity or NaN among them turns the
// rows before it into NaN (0 x inf).  Such rows are recomputed by these functions, which never touch a key behind them.  A row
// whose row sum, log-sum-exp or delta is NaN is not: it sees the NaN itself, and all of its results are NaN either way.
#pragma once

#include <math.h>

#include "po_common.h"

namespace po {

// acc[r] += w(jj) m[jj][lane + 64 r] over the n rows of m in order.  AHEAD rows are loaded before the first is used: a lone
// wave has no other to hide its loads behind (1: the vector kernels, which have).
template <typename T, int SLOTS, int AHEAD>
__device__ __forceinline__ void accumulate_weighted_rows(float (&acc)[SLOTS], float w, const T* __restrict__ m, int ld, int n,
                                                         int dh, int lane) {
  int jj = 0;
  if constexpr (AHEAD > 1)
    for (; jj + AHEAD <= n; jj += AHEAD) {
      float v[AHEAD][SLOTS];
#pragma unroll
      for (int u = 0; u < AHEAD; ++u)
#pragma unroll
        for (int r = 0; r < SLOTS; ++r) {
          int e = lane + kWave * r;
          v[u][r] = e < dh ? to_f32(m[(size_t)(jj + u) * ld + e]) : 0.f;
        }
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        float wj = __shfl(w, jj + u, kWave);
#pragma unroll
        for (int r = 0; r < SLOTS; ++r) acc[r] = fmaf(wj, v[u][r], acc[r]);
      }
    }
  for (; jj < n; ++jj) {
    float wj = __shfl(w, jj, kWave);
    const T* row = m + (size_t)jj * ld;
#pragma unroll
    for (int r = 0; r < SLOTS; ++r) {
      int e = lane + kWave * r;
      if (e < dh) acc[r] = fmaf(wj, to_f32(row[e]), acc[r]);
    }
  }
}

// Row i of head `head`: o_row[dh] and *lse.  query(e) is element e of the row's query, scaled; SLOTS * 64 >= dh, dh a multiple
// of AHEAD.  All 64 lanes of the wave call it with the same arguments.
template <typename T, int SLOTS, int AHEAD, typename Query>
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
      for (int e = 0; e < dh; e += AHEAD)
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) d = fmaf(query(e + u), to_f32(kr[e + u]), d);
      sc = d;
    }
    float mnew = fmaxf(m, wave_max(sc));
    float p = (j <= i) ? __expf(sc - mnew) : 0.f;
    float alpha = __expf(m - mnew);
    l = l * alpha + wave_sum(p);
#pragma unroll
    for (int r = 0; r < SLOTS; ++r) acc[r] *= alpha;
    accumulate_weighted_rows<T, SLOTS, AHEAD>(acc, p, vbase + (size_t)j0 * ld, ld, min(kWave, i - j0 + 1), dh, lane);
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
template <typename T, int SLOTS, int AHEAD, typename Query, typename Upstream>
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
      for (int e = 0; e < dh; e += AHEAD)
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
          sc = fmaf(query(e + u), to_f32(kr[e + u]), sc);
          dp = fmaf(upstream(e + u), to_f32(vr[e + u]), dp);
        }
      ds = __expf(sc - lse_i) * (dp - delta_i);
    }
    accumulate_weighted_rows<T, SLOTS, AHEAD>(acc, ds, kbase + (size_t)j0 * ld, ld, min(kWave, i - j0 + 1), dh, lane);
  }
#pragma unroll
  for (int r = 0; r < SLOTS; ++r) {
    int e = lane + kWave * r;
    if (e < dh) dq_row[e] = from_f32<T>(acc[r] * scale);
  }
}

__device__ __forceinline__ bool is_nan(float x) { return x != x; }

// ---- for the matrix-core kernels, whose waves own 32 rows with lane L holding part of row L % 32 -------------------
// The rows of which some lane says `bad`, one bit each, those from `rows` on left out.
__device__ __forceinline__ uint32_t rows_to_redo(bool bad, int rows) {
  const uint64_t b = __builtin_amdgcn_ballot_w64(bad);
  uint32_t m = __builtin_amdgcn_readfirstlane((uint32_t)b | (uint32_t)(b >> 32));
  return rows >= 32 ? m : rows <= 0 ? 0u : m & ((1u << rows) - 1u);
}

// A row of DH elements held by a wave, lane L elements L and L + 64; broadcast(e), e the same in every lane, hands element e to
// the active lanes.  It is called where only some are, so whatever it reads has to be made where all of them are: the
// registers are pinned there, and the choice between them is made on scalars.
template <int DH>
struct HeldRow {
  int v[DH > kWave ? 2 : 1];
  template <typename T>
  __device__ __forceinline__ HeldRow(const T* __restrict__ row, float factor, int lane) {
#pragma unroll
    for (int r = 0; r < (DH > kWave ? 2 : 1); ++r) {
      v[r] = __builtin_bit_cast(int, lane + kWave * r < DH ? to_f32(row[lane + kWave * r]) * factor : 0.f);
      asm volatile("" : "+v"(v[r]));
    }
  }
  __device__ __forceinline__ float broadcast(int e) const {
    int x = __builtin_amdgcn_readlane(v[0], e & (kWave - 1));
    if constexpr (DH > kWave) {
      const int y = __builtin_amdgcn_readlane(v[1], e & (kWave - 1));
      x = e < kWave ? x : y;
    }
    return __builtin_bit_cast(float, x);
  }
};

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
    const HeldRow<DH> q(qkv + (size_t)i * ld + head * DH, scale, lane);
    const T* k = qkv + h + (head / group) * DH;
    attention_forward_row<T, (DH + kWave - 1) / kWave, 8>([&](int e) { return q.broadcast(e); }, k, k + hkv, ld, i, dh, lane,
                                                          o + (size_t)i * h + head * DH, lse + (size_t)head * s + i);
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
    const HeldRow<DH> q(qkv + (size_t)i * ld + head * DH, scale, lane), g(d_o + (size_t)i * h + head * DH, 1.f, lane);
    const T* k = qkv + h + (head / group) * DH;
    attention_dq_row<T, (DH + kWave - 1) / kWave, 8>([&](int e) { return q.broadcast(e); },
                                                     [&](int e) { return g.broadcast(e); }, k, k + hkv, ld,
                                                     lse[(size_t)head * s + i], delta[(size_t)head * s + i], i, dh, lane,
                                                     scale, dqkv + (size_t)i * ld + head * DH);
  }
}

}  // namespace po
