// fp32 causal attention on the matrix cores (v_mfma_f32_32x32x2_f32: full fp32 products and sums), forward and
// backward, any sequence length, head sizes 32, 64, 96 and 128.
//
// What counts is that a SIMD has waves with MFMAs to issue (one takes 64 cycles, 2048 a product of two 32-row tiles over 64
// columns; two waves up to heads of 64, of whose blocks a CU's LDS holds two, one for heads of 96 and 128) and that no chain is long.  Every wave works on its own, no barrier in the loops: its two tiles of 32 keys (query
// rows) go HBM -> LDS directly into a place of its own, from which it reads 16-byte pieces of rows for the products over the head
// dimension and 32 consecutive floats of a row for the others.  (Read from global memory into registers instead, the compiler kept
// one or two loads in flight, a memory round trip per four MFMAs.)  A block owns only 32 rows (query rows in forward and dQ,
// keys in dK/dV) and its four waves split the tiles those meet, tile t to wave t % 4; the four partial results are added in
// wave order through LDS at the end (deterministic, no atomics).  Heaviest blocks of the causal triangle first; the backward is one
// launch, dK/dV blocks and then dQ blocks, which start where a light dK/dV block has ended.
//
// Rows of o and dQ whose sums are not finite, without a NaN of their own, are redone one by one (attention_rows.h), so that an infinity or NaN in a
// key or value reaches the rows at and behind it and no other.  What that costs where all is finite, one multiplication
// per sum, is not measurable (a stage of 16 heads of 64 at 1024 rows 4.07 and 4.05 ms).
//
// Layouts.  S^T = K Q^T puts the index a wave owns on the MFMA's column: lane L holds column L % 32 and rows
// 8 b + 4 (L / 32) + r (register 4 b + r).  Register e of such a tile is, as it stands, the second operand of step e of
// the product that follows (the step's two k-indices are the rows the two half-waves hold in register e), whose first
// operand is then 32 consecutive floats of row 8 b + 4 (L / 32) + r.  For the products over the head dimension a
// half-wave takes elements 8 kk + 4 (L / 32) + j in step (kk, j): a 16-byte load feeds four steps.
//
// s = 1024, 16 heads of 64: forward 27 us (42 with operands from global memory and blocks in plain order), backward 80 us (143 so and
// as two launches); s = 3000, 32 heads of 64: 317 (453) and 1055 us (1549; 7 s^2 h: 122 of 157 TFLOP/s); s = 2048, 32 heads of 128
// over 8: 340 (422) and 1130 us (2029); s = 128, 4 heads: 6.9 and 12 us (7.5 and 21.6), bound by the chain of one tile.  Asking for one of the two tiles
// of the next step while the other is still used gave nothing at 64 columns (registers spill) and 2 % at 128.
#include "attention_rows.h"
#include "mfma_common.h"

namespace po {

namespace {

constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ f32x16 mfma(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int e = 0; e < 16; ++e) z[e] = 0.f;
  return z;
}
// exp(x scale).  Two multiplications: with scale log2(e) as one constant its rounding is the same in every term of a row.
__device__ __forceinline__ float exp_scaled(float x, float scale) { return __builtin_amdgcn_exp2f(x * scale * kLog2e); }
// Row `row` of a matrix: this half-wave's 16-byte pieces.
template <int DH>
__device__ __forceinline__ void load_pieces(f32x4 (&f)[DH / 8], const float* row, int half) {
#pragma unroll
  for (int kk = 0; kk < DH / 8; ++kk) f[kk] = *reinterpret_cast<const f32x4*>(row + 8 * kk + 4 * half);
}

// A wave's copy of 32 rows of a matrix in LDS: piece c (16 bytes) of row r at place c ^ place_of(r), so that the reads of one
// piece of eight rows and of 32 floats of two rows that are four apart both fall into different banks.
template <int DH>
constexpr int kTileBytes = 32 * DH * 4;
template <int DH>
__device__ __forceinline__ int place_of(int row) {
  return (row & 7) ^ (DH % 64 == 0 ? ((row >> 2) & 1) << 3 : 0);
}
// Requests rows row0 .. row0 + 31 of the matrix at m (rows past `last`: the last one) into the tile at LDS byte `tile`.
template <int DH>
__device__ __forceinline__ void request_tile(unsigned tile, const float* m, int ld, int row0, int last, int lane) {
  const i32x4 buf = buffer_of(m + (size_t)row0 * ld, 0xffffffe0u);
  const int max_row = last - row0;
#pragma unroll
  for (int u = 0; u < kTileBytes<DH> / 1024; ++u) {
    const int byte = u * 1024 + lane * 16, row = byte / (DH * 4), c = (byte % (DH * 4) >> 4) ^ place_of<DH>(row);
    buffer_to_lds(tile + 1024u * u, (unsigned)min(row, max_row) * (unsigned)ld * 4 + c * 16, buf);
  }
}
// Where a lane reads in the first of a wave's two tiles; everything else is a constant offset from there.  (Left to itself the
// compiler keeps an address register per read, and spills.)
template <int DH>
struct LaneReads {
  static constexpr int PB = DH % 64 == 0 ? 8 : 4, RB = DH % 64 == 0 ? 2 : 1;
  int piece[PB];   // pieces 2 kk + lane / 32, kk < PB, of row lane % 32
  int row[4][RB];  // element 32 d + lane % 32, d < RB, of rows 4 (lane / 32) + r
  __device__ __forceinline__ LaneReads(int at, int lane) {
    const int half = lane >> 5, i = lane & 31;
#pragma unroll
    for (int k = 0; k < PB; ++k) {
      piece[k] = at + i * (DH * 4) + (((2 * k + half) ^ place_of<DH>(i)) << 4);
      asm volatile("" : "+v"(piece[k]));
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int d = 0; d < RB; ++d) {
        row[r][d] = at + (4 * half + r) * (DH * 4) + (((8 * d + (i >> 2)) ^ place_of<DH>(4 * half + r)) << 4) + (i & 3) * 4;
        asm volatile("" : "+v"(row[r][d]));
      }
  }
};
// c += rows of tile TILE times b over the head dimension.
template <int DH, int TILE>
__device__ __forceinline__ f32x16 dot_tile(const char* lds, const LaneReads<DH>& l, const f32x4 (&b)[DH / 8]) {
  constexpr int PB = LaneReads<DH>::PB;
  f32x16 c = zero16();
  auto piece = [&](int kk) {
    return *reinterpret_cast<const f32x4*>(lds + l.piece[kk % PB] + TILE * kTileBytes<DH> + kk / PB * PB * 32);
  };
  f32x4 a[2] = {piece(0), piece(1)};  // read two pieces ahead of their four MFMAs
#pragma unroll
  for (int kk = 0; kk < DH / 8; ++kk) {
    const f32x4 v = a[kk & 1];
    if (kk + 2 < DH / 8) a[kk & 1] = piece(kk + 2);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 4; ++j) c = mfma(v[j], b[kk][j], c);
  }
  return c;
}
// acc[d] += M^T w over the 32 rows of tile TILE: first operand rows of M, second w.
template <int DH, int TILE>
__device__ __forceinline__ void accumulate_rows(f32x16 (&acc)[DH / 32], const char* lds, const LaneReads<DH>& l,
                                                const f32x16& w) {
  constexpr int RB = LaneReads<DH>::RB, DT = DH / 32;
  auto element = [&](int e, int d) {
    return *reinterpret_cast<const float*>(lds + l.row[e & 3][d % RB] + TILE * kTileBytes<DH> + d / RB * RB * 128 +
                                           (e >> 2) * 8 * DH * 4);
  };
  constexpr int AHEAD = DT < 4 ? 3 : 2;  // a row is read that many steps ahead
  float a[4][DT];
#pragma unroll
  for (int e = 0; e < AHEAD; ++e)
#pragma unroll
    for (int d = 0; d < DT; ++d) a[e][d] = element(e, d);
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    if (e + AHEAD < 16)
#pragma unroll
      for (int d = 0; d < DT; ++d) a[(e + AHEAD) & 3][d] = element(e + AHEAD, d);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int d = 0; d < DT; ++d) acc[d] = mfma(a[e & 3][d], w[e], acc[d]);
  }
}
// A partial result of one wave in LDS: [register][lane].
template <int N>
__device__ __forceinline__ void put_partial(float* p, const f32x16 (&acc)[N], int lane) {
#pragma unroll
  for (int d = 0; d < N; ++d)
#pragma unroll
    for (int e = 0; e < 16; ++e) p[(d * 16 + e) * 64 + lane] = acc[d][e];
}
// The four waves' rows to redo, left in LDS before the barrier: all of them, and this wave's share (every fourth).
__device__ __forceinline__ uint32_t all_redo(const uint32_t* masks) {
  return __builtin_amdgcn_readfirstlane(masks[0] | masks[1] | masks[2] | masks[3]);
}
__device__ __forceinline__ uint32_t share_of(uint32_t redo, int wave) { return redo & (0x11111111u << wave); }
// Blocks by falling weight, of which every one finds a place at once: the first 256 go to a CU each, the next 256 to the same
// CUs in the same order, so every other such row is turned round: the heaviest block shares its CU with the lightest.
__device__ __forceinline__ int snake(int block, int blocks) {
  const int first = block & ~255;
  return first & 256 ? first + min(255, blocks - 1 - first) - (block - first) : block;
}

}  // namespace

template <int DH>
__global__ __launch_bounds__(256, 2) void attn_f32_fwd_kernel(const float* __restrict__ qkv, float* __restrict__ o,
                                                              float* __restrict__ lse, int s, int h, int hkv, int group,
                                                              float scale, int resident) {
  constexpr int DT = DH / 32, PART = 2 * kTileBytes<DH> / 4;
  // per wave a tile of K and one of V, later its partial output; then the waves' maxima and row sums, rows to redo
  extern __shared__ __align__(16) float lds[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  const int at = resident ? snake(blockIdx.x, gridDim.x) : (int)blockIdx.x, n_heads = h / DH;
  const int head = at % n_heads, q0 = ((int)gridDim.x - 1 - at) / n_heads * 32, q = q0 + (lane & 31);
  const int ld = h + 2 * hkv, last = s - 1;
  const float* kbase = qkv + h + (head / group) * DH;
  const float* vbase = kbase + hkv;
  const char* bytes = reinterpret_cast<const char*>(lds);
  const LaneReads<DH> reads(wave * PART * 4, lane);
  const unsigned k_lds = __builtin_amdgcn_readfirstlane((int)lds_byte(lds + wave * PART)), v_lds = k_lds + kTileBytes<DH>;
  const int n_tiles = min(q0 + 31, last) / 32 + 1;
  auto request = [&](int t) {
    request_tile<DH>(k_lds, kbase, ld, 32 * t, last, lane);
    request_tile<DH>(v_lds, vbase, ld, 32 * t, last, lane);
  };
  if (wave < n_tiles) request(wave);
  f32x4 qf[DH / 8];
  load_pieces<DH>(qf, qkv + (size_t)min(q, last) * ld + head * DH, half);
  f32x16 acc[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d) acc[d] = zero16();
  float m_run = -INFINITY, l_run = 0.f;
  for (int t = wave; t < n_tiles; t += 4) {
    wait_loads<0>();
    f32x16 p = dot_tile<DH, 0>(bytes, reads, qf);
    if (t == n_tiles - 1) {  // the tile of the diagonal; keys past s lie beyond it for every row there is
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (32 * t + 8 * (e >> 2) + 4 * half + (e & 3) > q) p[e] = -INFINITY;
    }
    float mx = m_run;
#pragma unroll
    for (int e = 0; e < 16; ++e) mx = fmaxf(mx, p[e]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float ref = mx == -INFINITY ? 0.f : mx;  // scores that are all -inf add nothing, instead of inf - inf
    float alpha = exp_scaled(m_run - ref, scale), sum = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      p[e] = exp_scaled(p[e] - ref, scale);
      sum += p[e];
    }
    m_run = mx;
    l_run = l_run * alpha + sum;
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[d][e] *= alpha;
    accumulate_rows<DH, 1>(acc, bytes, reads, p);
    wait_lds_reads();
    if (t + 4 < n_tiles) request(t + 4);
  }
  put_partial<DT>(lds + wave * PART, acc, lane);
  float* stat = lds + 4 * PART;
  uint32_t* redo_of = reinterpret_cast<uint32_t*>(stat + 8 * 64);
  const uint32_t redo_mine = rows_to_redo(not_finite<DT>(acc), s - q0);
  if (lane == 0) redo_of[wave] = redo_mine;
  stat[wave * 64 + lane] = m_run;
  stat[(4 + wave) * 64 + lane] = l_run + __shfl_xor(l_run, 32, 64);
  __syncthreads();
  // Wave w finishes registers 4 w .. 4 w + 3 (columns 32 d + 8 w + 4 half ..) of every lane's row.
  float m = stat[lane], f[4], l = 0.f;
#pragma unroll
  for (int w = 1; w < 4; ++w) m = fmaxf(m, stat[w * 64 + lane]);  // wave 0 has seen key 0: finite
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    f[w] = exp_scaled(stat[w * 64 + lane] - m, scale);
    l += stat[(4 + w) * 64 + lane] * f[w];
  }
  const uint32_t redo = all_redo(redo_of) & rows_to_redo(!is_nan(l), 32);
  if (redo) redo_forward_rows<float, DH>(share_of(redo, wave), q0, qkv, o, lse, s, h, hkv, group, head, scale);
  if (q > last || (redo >> (lane & 31) & 1)) return;
#pragma unroll
  for (int d = 0; d < DT; ++d) {
    f32x4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float x = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) x += lds[w * PART + (d * 16 + 4 * wave + r) * 64 + lane] * f[w];
      v[r] = x / l;
    }
    *reinterpret_cast<f32x4*>(o + (size_t)q * h + head * DH + 32 * d + 8 * wave + 4 * half) = v;
  }
  if (wave == 0 && half == 0) lse[(size_t)head * s + q] = fmaf(m, scale, __logf(l));
}

// Block `at` of heads * tiles, heaviest first: 32 query rows of a head.
template <int DH>
__device__ __forceinline__ void dq_block(float* lds, int at, const float* __restrict__ qkv, const float* __restrict__ d_o,
                                         const float* __restrict__ lse, const float* __restrict__ delta,
                                         float* __restrict__ dqkv, int s, int h, int hkv, int group, float scale) {
  constexpr int DT = DH / 32, PART = 2 * kTileBytes<DH> / 4;  // a wave's tiles of K and V, later its partial result
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  const int n_heads = h / DH, head = at % n_heads, q0 = ((s - 1) / 32 - at / n_heads) * 32, q = q0 + (lane & 31);
  const int ld = h + 2 * hkv, last = s - 1, qc = min(q, last);
  const float* kbase = qkv + h + (head / group) * DH;
  const float* vbase = kbase + hkv;
  const char* bytes = reinterpret_cast<const char*>(lds);
  const LaneReads<DH> reads(wave * PART * 4, lane);
  const unsigned k_lds = __builtin_amdgcn_readfirstlane((int)lds_byte(lds + wave * PART)), v_lds = k_lds + kTileBytes<DH>;
  const int n_tiles = min(q0 + 31, last) / 32 + 1;
  auto request = [&](int t) {
    request_tile<DH>(k_lds, kbase, ld, 32 * t, last, lane);
    request_tile<DH>(v_lds, vbase, ld, 32 * t, last, lane);
  };
  if (wave < n_tiles) request(wave);
  f32x4 qf[DH / 8], dof[DH / 8];
  load_pieces<DH>(qf, qkv + (size_t)qc * ld + head * DH, half);
  load_pieces<DH>(dof, d_o + (size_t)qc * h + head * DH, half);
  const float lse_q = lse[(size_t)head * s + qc], delta_q = delta[(size_t)head * s + qc];
  f32x16 dq[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d) dq[d] = zero16();
  for (int t = wave; t < n_tiles; t += 4) {
    wait_loads<0>();
    f32x16 p = dot_tile<DH, 0>(bytes, reads, qf);
    f32x16 ds = dot_tile<DH, 1>(bytes, reads, dof);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      float pe = __builtin_amdgcn_exp2f(fmaf(p[e], scale, -lse_q) * kLog2e);
      if (t == n_tiles - 1 && 32 * t + 8 * (e >> 2) + 4 * half + (e & 3) > q) pe = 0.f;
      ds[e] = pe * (ds[e] - delta_q);
    }
    accumulate_rows<DH, 0>(dq, bytes, reads, ds);
    wait_lds_reads();
    if (t + 4 < n_tiles) request(t + 4);
  }
  put_partial<DT>(lds + wave * PART, dq, lane);
  uint32_t* redo_of = reinterpret_cast<uint32_t*>(lds + 4 * PART);
  const uint32_t redo_mine = rows_to_redo(not_finite<DT>(dq) && !is_nan(lse_q + delta_q), s - q0);
  if (lane == 0) redo_of[wave] = redo_mine;
  __syncthreads();
  const uint32_t redo = all_redo(redo_of);
  if (redo) redo_dq_rows<float, DH>(share_of(redo, wave), q0, qkv, d_o, lse, delta, dqkv, s, h, hkv, group, head, scale);
  if (q > last || (redo >> (lane & 31) & 1)) return;
#pragma unroll
  for (int d = 0; d < DT; ++d) {
    f32x4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float x = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) x += lds[w * PART + (d * 16 + 4 * wave + r) * 64 + lane];
      v[r] = x * scale;
    }
    *reinterpret_cast<f32x4*>(dqkv + (size_t)q * ld + head * DH + 32 * d + 8 * wave + 4 * half) = v;
  }
}

// Block `at` of key/value heads * tiles, heaviest first: 32 keys of one key/value head; its waves walk the query tiles of
// every query head that reads it.
template <int DH>
__device__ __forceinline__ void dkv_block(float* lds, int at, const float* __restrict__ qkv, const float* __restrict__ d_o,
                                          const float* __restrict__ lse, const float* __restrict__ delta,
                                          float* __restrict__ dqkv, int s, int h, int hkv, int group, float scale) {
  constexpr int DT = DH / 32, PART = kTileBytes<DH> / 4;  // a wave's tiles of Q and dO, later its partial results
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  const int n_kv = hkv / DH, kv_head = at % n_kv, first = at / n_kv, key = first * 32 + (lane & 31);
  const int ld = h + 2 * hkv, last = s - 1;
  const char* bytes = reinterpret_cast<const char*>(lds);
  const LaneReads<DH> reads(wave * 2 * PART * 4, lane);
  const unsigned q_lds = __builtin_amdgcn_readfirstlane((int)lds_byte(lds + wave * 2 * PART)), do_lds = q_lds + kTileBytes<DH>;
  const int n_q = last / 32 + 1 - first, n_it = group * n_q;
  auto request = [&](int it) {
    const int g = it / n_q, q0 = (first + it - g * n_q) * 32, head = kv_head * group + g;
    request_tile<DH>(q_lds, qkv + head * DH, ld, q0, last, lane);
    request_tile<DH>(do_lds, d_o + head * DH, h, q0, last, lane);
  };
  if (wave < n_it) request(wave);
  f32x4 kf[DH / 8], vf[DH / 8];
  const float* krow = qkv + (size_t)min(key, last) * ld + h + kv_head * DH;
  load_pieces<DH>(kf, krow, half);
  load_pieces<DH>(vf, krow + hkv, half);
  f32x16 dk[DT], dv[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d) dk[d] = dv[d] = zero16();
  for (int it = wave; it < n_it; it += 4) {
    const int g = it / n_q, q0 = (first + it - g * n_q) * 32, head = kv_head * group + g;
    // lse of row lane % 32 in the lower half-wave, its delta in the upper
    const float stat = (half ? delta : lse)[(size_t)head * s + min(q0 + (lane & 31), last)];
    wait_loads<0>();
    f32x16 p = dot_tile<DH, 0>(bytes, reads, kf);
    f32x16 ds = dot_tile<DH, 1>(bytes, reads, vf);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int row = 8 * (e >> 2) + 4 * half + (e & 3);
      p[e] = __builtin_amdgcn_exp2f(fmaf(p[e], scale, -__shfl(stat, row, 64)) * kLog2e);
      ds[e] = p[e] * (ds[e] - __shfl(stat, 32 + row, 64));
    }
    if (q0 == first * 32 || q0 + 31 > last) {  // the diagonal, or rows past the end
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int q = q0 + 8 * (e >> 2) + 4 * half + (e & 3);
        // dS is selected too: 0 times the dP of a row that is not finite is no 0
        if (q > last || key > q) p[e] = ds[e] = 0.f;
      }
    }
    accumulate_rows<DH, 1>(dv, bytes, reads, p);
    accumulate_rows<DH, 0>(dk, bytes, reads, ds);
    wait_lds_reads();
    if (it + 4 < n_it) request(it + 4);
  }
  put_partial<DT>(lds + wave * 2 * PART, dk, lane);
  put_partial<DT>(lds + wave * 2 * PART + PART, dv, lane);
  __syncthreads();
  if (key > last) return;
  float* out = dqkv + (size_t)key * ld + h + kv_head * DH + 8 * wave + 4 * half;
#pragma unroll
  for (int d = 0; d < DT; ++d) {
    f32x4 vk, vv;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float x = 0.f, y = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        x += lds[w * 2 * PART + (d * 16 + 4 * wave + r) * 64 + lane];
        y += lds[w * 2 * PART + PART + (d * 16 + 4 * wave + r) * 64 + lane];
      }
      vk[r] = x * scale;
      vv[r] = y;
    }
    *reinterpret_cast<f32x4*>(out + 32 * d) = vk;
    *reinterpret_cast<f32x4*>(out + hkv + 32 * d) = vv;
  }
}

template <int DH>
__global__ __launch_bounds__(256, DH > 64 ? 1 : 2) void attn_f32_bwd_kernel(const float* __restrict__ qkv, const float* __restrict__ d_o,
                                                              const float* __restrict__ lse, const float* __restrict__ delta,
                                                              float* __restrict__ dqkv, int s, int h, int hkv, int group,
                                                              float scale, int dkv_blocks) {
  extern __shared__ __align__(16) float lds[];
  // the dQ blocks take over the CUs of light dK/dV blocks while the heavy ones are still at work
  if ((int)blockIdx.x < dkv_blocks)
    dkv_block<DH>(lds, blockIdx.x, qkv, d_o, lse, delta, dqkv, s, h, hkv, group, scale);
  else
    dq_block<DH>(lds, blockIdx.x - dkv_blocks, qkv, d_o, lse, delta, dqkv, s, h, hkv, group, scale);
}
// delta[head][row] = dO . O of that row and head: eight lanes a row, 16 bytes of both per lane and step, added as a tree: with a
// lane's products one after the other heads of 128 were 8.8e-8 from 64 bits, with the tree 7.3e-8 (the kernel of any head size,
// a wave per row, too).
template <int DH>
__global__ __launch_bounds__(256) void attn_f32_delta_kernel(const float* __restrict__ o, const float* __restrict__ d_o,
                                                             float* __restrict__ delta, int s, int h) {
  const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
  const int n_heads = h / DH, part = threadIdx.x & 7;
  const size_t pair = t >> 3, row = pair / n_heads;  // (row, head), heads fastest: in address order
  const int head = (int)(pair - row * n_heads);
  constexpr int N = DH / 32;
  float v[N] = {};
  if (row < (size_t)s) {
    const size_t at = row * h + head * DH + part * 4;
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const f32x4 a = *reinterpret_cast<const f32x4*>(o + at + 32 * u), b = *reinterpret_cast<const f32x4*>(d_o + at + 32 * u);
      v[u] = fmaf(a[0], b[0], a[1] * b[1]) + fmaf(a[2], b[2], a[3] * b[3]);
    }
  }
#pragma unroll
  for (int u = 0; u + 1 < N; u += 2) v[u] += v[u + 1];
  float d = v[0];
  if constexpr (N > 2) d += v[2];
#pragma unroll
  for (int m = 1; m < 8; m <<= 1) d += __shfl_xor(d, m);
  if (part == 0 && row < (size_t)s) delta[(size_t)head * s + row] = d;
}

// ---- host side -------------------------------------------------------------------------------------------------
bool attention_f32_supported(const void* qkv, const void* o, int s, int h, int n_heads, int n_kv_heads) {
  if (s <= 0 || h <= 0 || n_heads <= 0 || h % n_heads != 0 || n_kv_heads <= 0 || n_heads % n_kv_heads != 0) return false;
  if (s > 32 * kMaxGridY) return false;
  // the backward's blocks, 256 threads each, in one dimension of a grid
  if (((int64_t)n_heads + n_kv_heads) * ceil_div(s, 32) >= (int64_t)1 << 24) return false;
  const int dh = h / n_heads;
  // a lane's offset in a tile of 32 rows fits 32 bits
  if (((int64_t)h + 2 * (int64_t)n_kv_heads * dh) * (4 * 32) > (int64_t)1 << 32) return false;
  return (dh == 32 || dh == 64 || dh == 96 || dh == 128) && ((uintptr_t)qkv | (uintptr_t)o) % 16 == 0;
}

template <int DH>
static bool forward_f32(const float* qkv, float* o, float* lse, int s, int h, int n_heads, int n_kv_heads,
                        hipStream_t stream) {
  constexpr int smem = 8 * kTileBytes<DH> + (8 * 64 + 4) * 4;
  static LdsLimit lds;
  if (!lds.allow(attn_f32_fwd_kernel<DH>, smem)) return false;
  // two blocks fit the LDS of a CU up to heads of 64 columns
  const int blocks = n_heads * ceil_div(s, 32);
  attn_f32_fwd_kernel<DH><<<blocks, 256, smem, stream>>>(qkv, o, lse, s, h, n_kv_heads * DH, n_heads / n_kv_heads,
                                                         1.0f / sqrtf((float)DH), DH <= 64 && blocks <= 512);
  return launch_ok("attn_f32_fwd_kernel");
}

template <int DH>
static bool backward_f32(const float* qkv, const float* lse, const float* delta, const float* d_o, float* dqkv, int s,
                         int h, int n_heads, int n_kv_heads, hipStream_t stream) {
  constexpr int smem = 8 * kTileBytes<DH> + 16;
  static LdsLimit lds;
  if (!lds.allow(attn_f32_bwd_kernel<DH>, smem)) return false;
  const int hkv = n_kv_heads * DH, group = n_heads / n_kv_heads;
  const float scale = 1.0f / sqrtf((float)DH);
  const int tiles = ceil_div(s, 32);
  attn_f32_bwd_kernel<DH><<<(n_kv_heads + n_heads) * tiles, 256, smem, stream>>>(qkv, d_o, lse, delta, dqkv, s, h, hkv,
                                                                              group, scale, n_kv_heads * tiles);
  return launch_ok("attn_f32_bwd_kernel");
}

bool attention_forward_f32(const float* qkv, float* o, float* lse, int s, int h, int n_heads, int n_kv_heads,
                           hipStream_t stream) {
  switch (h / n_heads) {
    case 32: return forward_f32<32>(qkv, o, lse, s, h, n_heads, n_kv_heads, stream);
    case 64: return forward_f32<64>(qkv, o, lse, s, h, n_heads, n_kv_heads, stream);
    case 96: return forward_f32<96>(qkv, o, lse, s, h, n_heads, n_kv_heads, stream);
    default: return forward_f32<128>(qkv, o, lse, s, h, n_heads, n_kv_heads, stream);
  }
}

bool attention_backward_f32(const float* qkv, const float* lse, const float* delta, const float* d_o, float* dqkv, int s,
                            int h, int n_heads, int n_kv_heads, hipStream_t stream) {
  switch (h / n_heads) {
    case 32: return backward_f32<32>(qkv, lse, delta, d_o, dqkv, s, h, n_heads, n_kv_heads, stream);
    case 64: return backward_f32<64>(qkv, lse, delta, d_o, dqkv, s, h, n_heads, n_kv_heads, stream);
    case 96: return backward_f32<96>(qkv, lse, delta, d_o, dqkv, s, h, n_heads, n_kv_heads, stream);
    default: return backward_f32<128>(qkv, lse, delta, d_o, dqkv, s, h, n_heads, n_kv_heads, stream);
  }
}

bool attention_delta_f32(const float* o, const float* d_o, float* delta, int s, int h, int n_heads, hipStream_t stream) {
  const unsigned blocks = (unsigned)(((size_t)s * n_heads * 8 + 255) / 256);
  switch (h / n_heads) {
    case 32: attn_f32_delta_kernel<32><<<blocks, 256, 0, stream>>>(o, d_o, delta, s, h); break;
    case 64: attn_f32_delta_kernel<64><<<blocks, 256, 0, stream>>>(o, d_o, delta, s, h); break;
    case 96: attn_f32_delta_kernel<96><<<blocks, 256, 0, stream>>>(o, d_o, delta, s, h); break;
    default: attn_f32_delta_kernel<128><<<blocks, 256, 0, stream>>>(o, d_o, delta, s, h);
  }
  return launch_ok("attn_f32_delta_kernel");
}

}  // namespace po
