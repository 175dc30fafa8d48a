// What the matrix-core GEMMs with small tiles share (gemm_small.hip, gemm_f32.hip): an operand's chunk of K on its way into
// LDS, fragments out of it, the epilogue on one vector, a tile's place.
#pragma once

#include "column_sums.h"
#include "mfma_common.h"

namespace po {

template <typename T> struct MfmaOf;
template <> struct MfmaOf<float> {
  static constexpr int KU = 32;  // k per chunk of 128 bytes
};
template <> struct MfmaOf<bf16> {
  static constexpr int KU = 64;
};

// ---- one operand's chunk in LDS ------------------------------------------------------------------------------
// KMAJOR == false: [R rows][128 bytes], 16-byte piece c of row r at c ^ (r & 7).
// KMAJOR == true: [KU k][R elements].  bf16: 32-byte unit u of row k at u ^ (k & mask), as the transposing reads like
// it; fp32: 16-byte piece c at c ^ 8 for odd groups of four k, so that the two half-waves (k and k + 4) hit different
// banks; with 16 elements a row k moves within its group of four instead, by the group's number, so that a wave's four k
// (4 g + j) do.
template <typename T, int R, bool KMAJOR>
struct Operand {
  static constexpr int E = sizeof(T), KU = MfmaOf<T>::KU;
  static constexpr int BYTES = R * 128;
  static constexpr int LOADS = BYTES / 1024;
  static constexpr int ROW_BYTES = R * E;  // KMAJOR
  unsigned voff[LOADS];
  const char* base;       // tile row 0, first k of this wave's next chunk
  int64_t left;           // bytes from base to the end of the operand
  int64_t step;           // from one chunk of this wave to its next

  __device__ __forceinline__ static int piece_of(int pos16, int k) {  // which 16-byte piece of row k lies at pos16
    if (E == 2) {
      constexpr int MASK = R >= 128 ? 7 : R / 16 - 1;
      return (((pos16 >> 1) ^ (k & MASK)) << 1) | (pos16 & 1);
    }
    return R >= 64 ? pos16 ^ (((k >> 2) & 1) << 3) : pos16;
  }

  static constexpr bool TURNED = KMAJOR && E == 4 && R == 16;
  __device__ __forceinline__ static int slot_of(int k) { return TURNED ? (k & ~3) | ((k + (k >> 2)) & 3) : k; }

  // p: the operand; ld in elements; row0: first row of the tile (of `rows`); chunk: this wave's first chunk of K.
  __device__ __forceinline__ void init(const T* p, int ld, int row0, int rows, int K, int chunk, int chunk_step, int lane) {
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
      int byte = u * 1024 + lane * 16;
      if (!KMAJOR) {
        int row = byte >> 7, c = ((byte >> 4) & 7) ^ (row & 7);
        voff[u] = (unsigned)row * (unsigned)ld * E + c * 16;
      } else {
        const int slot = byte / ROW_BYTES, k = TURNED ? (slot & ~3) | ((slot - (slot >> 2)) & 3) : slot;
        const int c = piece_of((byte % ROW_BYTES) >> 4, k);
        voff[u] = (unsigned)k * (unsigned)ld * E + c * 16;
      }
    }
    int64_t first = KMAJOR ? (int64_t)chunk * KU * ld + row0 : (int64_t)row0 * ld + (int64_t)chunk * KU;
    int64_t end = KMAJOR ? (int64_t)(K - 1) * ld + rows : (int64_t)(rows - 1) * ld + K;
    base = reinterpret_cast<const char*>(p) + first * E;
    left = (end - first) * E;
    step = (int64_t)chunk_step * (KMAJOR ? (int64_t)KU * ld * E : 128);
  }
  // Requests the chunk at `base` into LDS at `lds`; k_left: how many k the chunk has (>= KU: all of them; <= 0: none, the
  // stage gets zeros).
  __device__ __forceinline__ void issue(unsigned lds, int k_left, int lane) {
    i32x4 buf = buffer_of(base, (unsigned)min(max(left, (int64_t)0), (int64_t)0xffffffe0));
    if (!KMAJOR && k_left < KU) {  // the last chunk of a K that is no multiple of KU
#pragma unroll
      for (int u = 0; u < LOADS; ++u) {
        int byte = u * 1024 + lane * 16;
        int c = ((byte >> 4) & 7) ^ ((byte >> 7) & 7);
        buffer_to_lds(lds + 1024u * u, c * (16 / E) < k_left ? voff[u] : kOutOfBuffer, buf);
      }
    } else {
#pragma unroll
      for (int u = 0; u < LOADS; ++u) buffer_to_lds(lds + 1024u * u, voff[u], buf);
    }
    base += step;
    left -= step;
  }
};

// Fragment of 32 rows (row0 + lane % 32) for kk: bf16: k = 16 kk + 8 (lane / 32) + 0..7 (one MFMA); fp32:
// k = 8 kk + 4 (lane / 32) + 0..3 (four MFMAs).
template <int R, bool KMAJOR>
__device__ __forceinline__ bf16x8 fragment(const bf16*, const char* lds, int row0, int kk, int lane) {
  if (!KMAJOR) {
    int row = row0 + (lane & 31);
    return *reinterpret_cast<const bf16x8*>(lds + row * 128 + (((2 * kk + (lane >> 5)) ^ (row & 7)) << 4));
  }
  // transposing read: lane r of a group of 16 supplies row k0 + r / 4, columns 4 (r % 4) .. + 3; lane i receives
  // k0 .. k0 + 3 of column i
  constexpr int MASK = R >= 128 ? 7 : R / 16 - 1;
  typedef s16x4 __attribute__((address_space(3)))* lds_ptr;
  int i = lane & 15, grp = lane >> 4;
  int m = row0 + 16 * (grp & 1) + 4 * (i & 3);
  int k = 16 * kk + 8 * (grp >> 1) + (i >> 2);
  const char* p0 = lds + k * (2 * R) + (((m >> 4) ^ (k & MASK)) << 5) + (m & 15) * 2;
  const char* p1 = lds + (k + 4) * (2 * R) + (((m >> 4) ^ ((k + 4) & MASK)) << 5) + (m & 15) * 2;
  union {
    s16x4 h[2];
    bf16x8 v;
  } u;
  u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)p0);
  u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)p1);
  return u.v;
}
template <int R, bool KMAJOR>
__device__ __forceinline__ f32x4 fragment(const float*, const char* lds, int row0, int kk, int lane) {
  if (!KMAJOR) {
    int row = row0 + (lane & 31);
    return *reinterpret_cast<const f32x4*>(lds + row * 128 + (((2 * kk + (lane >> 5)) ^ (row & 7)) << 4));
  }
  int k = 8 * kk + 4 * (lane >> 5), row = row0 + (lane & 31);
  int at = R >= 64 ? (((row >> 2) ^ ((lane >> 5) << 3)) << 4) + (row & 3) * 4 : row * 4;
  f32x4 v;
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = *reinterpret_cast<const float*>(lds + (k + j) * (4 * R) + at);
  return v;
}
// Fragment of 16 rows for kk: k = 16 kk + 4 (lane / 16) + 0..3 of row lane % 16, four MFMAs of 16 x 16 x 4.
template <bool KMAJOR>
__device__ __forceinline__ f32x4 fragment16(const char* lds, int kk, int lane) {
  const int row = lane & 15, g = lane >> 4;
  if (!KMAJOR) return *reinterpret_cast<const f32x4*>(lds + row * 128 + (((4 * kk + g) ^ (row & 7)) << 4));
  f32x4 v;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    v[j] = *reinterpret_cast<const float*>(lds + Operand<float, 16, true>::slot_of(16 * kk + 4 * g + j) * 64 + row * 4);
  return v;
}
// C^T-wise product: the B fragment goes into the first slot, so a lane holds four consecutive n of one row m.
__device__ __forceinline__ f32x16 multiply(bf16x8 b, bf16x8 a, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 multiply(f32x4 b, f32x4 a, f32x16 c) {
#pragma unroll
  for (int j = 0; j < 4; ++j) c = __builtin_amdgcn_mfma_f32_32x32x2f32(b[j], a[j], c, 0, 0, 0);
  return c;
}

// ---- epilogue on V consecutive n of row m, all inside the result and 16-byte aligned ---------------------------
template <typename T>
__device__ __forceinline__ void epilogue_vector(const Epilogue& e, int m, int n, float* a) {
  constexpr int V = Vec16<T>::N;
  size_t idx = (size_t)m * e.ldc + n;
  if (e.acc_f32) {
#pragma unroll
    for (int i = 0; i < V; i += 4) {
      f32x4* p = reinterpret_cast<f32x4*>(e.acc_f32 + idx + i);
      f32x4 v = {a[i], a[i + 1], a[i + 2], a[i + 3]};
      *p = *p + v;
    }
    return;
  }
  if (e.bias) {
    Vec16<T> b = load16(static_cast<const T*>(e.bias) + n);
#pragma unroll
    for (int i = 0; i < V; ++i) a[i] += to_f32(b.v[i]);
  }
  if (e.residual) {
    Vec16<T> r = load16(static_cast<const T*>(e.residual) + idx);
#pragma unroll
    for (int i = 0; i < V; ++i) a[i] += to_f32(r.v[i]);
  }
  Vec16<T> o, g;
  if (e.gelu_u) {
    Vec16<T> u = load16(static_cast<const T*>(e.gelu_u) + idx);
#pragma unroll
    for (int i = 0; i < V; ++i) {
      float gf, dgf;
      gelu_and_grad_f(to_f32(u.v[i]), gf, dgf);
      g.v[i] = from_f32<T>(gf);
      o.v[i] = from_f32<T>(a[i] * dgf);
    }
  } else {
#pragma unroll
    for (int i = 0; i < V; ++i) o.v[i] = from_f32<T>(a[i]);
    if (e.gelu_out) {
#pragma unroll
      for (int i = 0; i < V; ++i) g.v[i] = from_f32<T>(gelu_f(to_f32(o.v[i])));
    }
  }
  if (e.out) store16(static_cast<T*>(e.out) + idx, o);
  if (e.gelu_out) store16(static_cast<T*>(e.gelu_out) + idx, g);
}

struct SmallProblem {
  const void* A;
  const void* B;
  Epilogue ep;
  int M, N, K, lda, ldb;
  int tiles_n, first_tile;  // of the launch's tiles
  int vec;                  // every row of the result and its operands starts on a 16-byte boundary
};

constexpr int kMaxSmallRows = 128;  // of an operand's tile: the largest row or k whose offset a lane forms is one less
constexpr int kMaxSmallGroup = 4;
struct SmallGroup {
  SmallProblem p[kMaxSmallGroup];
  int n, tiles;  // tiles: of all of them (set by gemm_f32.hip, whose grid may have blocks without one)
};
// Tiles in groups of eight rows, so that a run of them is compact in both dimensions.
__device__ __forceinline__ void place_of_tile(int tile, int tiles_m, int tiles_n, int& m, int& n) {
  const int first = tile / (8 * tiles_n) * 8, rows = min(tiles_m - first, 8), at = tile - first * tiles_n;
  m = first + at % rows;
  n = at / rows;
}

// Column sums that a group's launch does beside its products, in its first `blocks` blocks.
struct GroupSums {
  ReduceBatch batch;
  int rows, blocks;
};

// Block ids equal modulo 8 share an XCD: each XCD gets a run of neighbouring tiles (and their operands its L2).  The first
// `before` blocks have no tile.
__device__ __forceinline__ int tile_of_block(int before = 0) {
  const int n = gridDim.x - before, pid = blockIdx.x - before;
  return n % 8 == 0 ? (pid % 8) * (n / 8) + pid / 8 : pid;
}

// gemm_f32.hip: fp32 problems whose operands gemm_small has checked.
bool gemm_f32(int trans_a, int trans_b, SmallProblem& p, hipStream_t stream);
bool gemm_f32_grouped(SmallGroup& g, const GroupSums* sums, hipStream_t stream);
dim3 gemm_f32_grid(int64_t tiles, int threads);
int gemm_f32_form(int n, const int* M, const int* N, int K);  // 0: 32 x 64 tiles, 1: 64 x 64, 2: 128 x 64

}  // namespace po
