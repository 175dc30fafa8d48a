// What the bf16 attention kernels share: a tile of rows in LDS, the fragments that MFMAs take from it, probabilities (and dS)
// as an operand.
#pragma once

#include "mfma_common.h"

namespace po {

#define LDS_AS3(p) ((s16x4 __attribute__((address_space(3)))*)(p))

// ---- LDS tile --------------------------------------------------------------------
// [rows][DH] bf16, unpadded: the 16-byte chunk c of row r sits at chunk position c ^ swz(r).
// One tile serves both kinds of MFMA operand reads without bank conflicts:
//  * ds_read_b128 "row" fragments (contraction over the head dimension): 16 lanes read the same
//    chunk of 16 consecutive rows; swz is a bijection of those rows onto the 16 chunk positions
//    of a 256-byte bank line (for DH = 64 two rows share a line and the row parity picks the half);
//  * transposing reads (contraction over the tile's rows): a half-wave reads 64 contiguous bytes
//    of four consecutive rows; swz sends them to the four different 64-byte quarters of a line.
template <int DH>
__device__ __forceinline__ int swz(int r) {
  if (DH == 128) return ((r & 3) << 2) | ((r >> 2) & 3);
  return (((r >> 1) & 1) << 2) | ((r >> 2) & 3);
}
template <int DH>
__device__ __forceinline__ int tile_offset(int row, int chunk) {
  return row * (DH * 2) + ((chunk ^ swz<DH>(row)) << 4);
}
// Fragment whose contraction index is the tile's row: lane (column c = lane % 32 of the
// 32-wide block starting at col0, half = lane / 32) receives rows
// {row0 + 4 half + 0..3} and {row0 + 4 half + 8 + 0..3} of column col0 + c.
// Within a group of 16 lanes, the transposing read hands lane i element (i % 4) of the
// four addresses supplied by lanes i / 4, 4 + i / 4, 8 + i / 4, 12 + i / 4 of the group.
template <int DH>
__device__ __forceinline__ bf16x8 read_tr_fragment(const char* tile, int row0, int col0, int lane) {
  int i = lane & 15;
  int grp = lane >> 4;
  int half = grp >> 1;
  int r = row0 + 4 * half + (i >> 2);
  int c = col0 + 16 * (grp & 1) + 4 * (i & 3);
  int inner = (c & 7) * 2;
  s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_AS3(tile + tile_offset<DH>(r, c >> 3) + inner));
  s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_AS3(tile + tile_offset<DH>(r + 8, c >> 3) + inner));
  union {
    struct {
      s16x4 a, b;
    } s;
    bf16x8 v;
  } u;
  u.s.a = lo;
  u.s.b = hi;
  return u.v;
}

template <int DH>
__device__ __forceinline__ bf16x8 read_row_fragment(const char* tile, int row, int chunk) {
  return *reinterpret_cast<const bf16x8*>(tile + tile_offset<DH>(row, chunk));
}

// Eight consecutive accumulator values -> bf16 operand fragment.
__device__ __forceinline__ bf16x8 pack_bf16x8(const f32x16& a, int first) {
  bf16x8 r;
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = (bf16)a[first + e];
  return r;
}

// Eight probabilities (or dS) as an operand: rounded to bf16 once, or (FULL) as the sum of three bf16 terms that is the
// fp32 value itself: its upper 16 bits, those of what is left, and the rest, which has no more than eight significant bits.
// Both differences are exact.
template <bool FULL>
struct Weights {
  bf16x8 term[FULL ? 3 : 1];
};
// Pair p of the eight values: upper halves of two floats side by side in one register of each term.
__device__ __forceinline__ void split_pair(Weights<true>& w, const f32x16& a, int first, int p) {
  float x0 = a[first + 2 * p], x1 = a[first + 2 * p + 1];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const unsigned u0 = __builtin_bit_cast(unsigned, x0), u1 = __builtin_bit_cast(unsigned, x1);
    u32x4 v = __builtin_bit_cast(u32x4, w.term[k]);
    v[p] = __builtin_amdgcn_perm(u1, u0, 0x07060302);
    w.term[k] = __builtin_bit_cast(bf16x8, v);
    x0 -= __builtin_bit_cast(float, u0 & 0xffff0000u);
    x1 -= __builtin_bit_cast(float, u1 & 0xffff0000u);
  }
}
template <bool FULL>
__device__ __forceinline__ Weights<FULL> weights_of(const f32x16& a, int first) {
  Weights<FULL> w;
  if constexpr (FULL) {
#pragma unroll
    for (int p = 0; p < 4; ++p) split_pair(w, a, first, p);
  } else {
    w.term[0] = pack_bf16x8(a, first);
  }
  return w;
}
// c += m^T w, the small terms first.
template <bool FULL>
__device__ __forceinline__ f32x16 multiply(const bf16x8& m, const Weights<FULL>& w, f32x16 c) {
  if constexpr (FULL) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(m, w.term[2], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(m, w.term[1], c, 0, 0, 0);
  }
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(m, w.term[0], c, 0, 0, 0);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

}  // namespace po
