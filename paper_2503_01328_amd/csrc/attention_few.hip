// bf16 causal attention on the matrix cores for launches of few rows, forward and backward: those whose blocks of 128 rows
// (attention_mfma.hip) would leave most CUs without one, where a launch is the chain of its longest block and little else.
//
// A block owns only 32 rows (query rows in forward and dQ, keys in dK/dV) and its waves split the tiles of 32 keys (query rows)
// those meet, tile t to wave t % W; every wave has a stage or two of its own, HBM -> LDS directly, and no barrier until the
// partial results are added in wave order through LDS (deterministic, no atomics).  Against a 128-row block of eight waves that is
// a quarter of the tiles per wave, at four times the tile loads per row.  Heaviest blocks of the causal triangle first; the
// backward is one launch, dK/dV blocks and then dQ blocks.  8 heads of 64 at 512 rows: forward 8.9 -> 5.8 us, backward with delta
// 17.0 -> 9.9; a stage of them (width 512, 2 layers, 4 microbatches) 1009 -> 917 us.  Bound by launch, first load and the merge: one
// tile a wave (128 rows) takes 4.0 and 7.1 us.  A dK/dV block walks all query heads of its key/value head, or
// hpb of them with fp32 partial results in a workspace that attn_group_sum_kernel adds up.
//
// Operand layouts, the three-term weights of sequences that are no multiple of 128 (EDGE) and what happens to rows that are
// not finite are those of attention_mfma.hip; without EDGE a non-finite key or value reaches the rows before it in its tile
// of 32.
#include <algorithm>

#include "attention_rows.h"
#include "attention_tile.h"

namespace po {

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kRows = 32;  // of a tile and of a block

// Waves of a block, their stages, bytes of a tile and of a stage (two tiles), and where in LDS what follows the stages begins.  Heads
// of 128 need more than 256 registers in the backward: one wave per SIMD.  In the forward they have eight waves too, for which LDS has
// room for one stage each: the next K is requested once the scores are formed, the next V behind the product (four waves of two
// stages / this, us: 100 rows, 16 heads 6.1 / 5.6, 512 rows, 8 heads 9.0 / 8.6, 777 rows, 10 heads 15.2 / 12.0, 4096 rows, 2 heads 40.6 / 28.7).
template <int DH, bool FORWARD = false>
struct Few {
  static constexpr int W = DH == 64 || FORWARD ? 8 : 4, NS = DH == 64 || !FORWARD ? 2 : 1, TILE = kRows * DH * 2, STAGE = 2 * TILE, LOADS = TILE / 1024;
  static constexpr int AFTER = W * NS * STAGE;
};

__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int e = 0; e < 16; ++e) z[e] = 0.f;
  return z;
}

// A wave's loads of a tile of 32 rows that are ld elements apart: the byte offset of a lane's 16 bytes in each of them.
template <int DH>
struct TileLoads {
  unsigned off[Few<DH>::LOADS];
  __device__ __forceinline__ TileLoads(int ld, int lane) {
#pragma unroll
    for (int u = 0; u < Few<DH>::LOADS; ++u) {
      const int byte = u * 1024 + lane * 16, row = byte / (DH * 2), c = (byte % (DH * 2) >> 4) ^ swz<DH>(row);
      off[u] = (unsigned)row * (unsigned)ld * 2u + c * 16;
    }
  }
  // Rows row0 .. row0 + 31 of the matrix at m into the tile at LDS byte `tile`; rows from s on become zeros.
  __device__ __forceinline__ void request(unsigned tile, const bf16* m, int ld, int row0, int s) const {
    const int rows = min(s - row0, kRows);  // at least one
    const i32x4 buf = buffer_of(m + (size_t)row0 * ld, ((unsigned)(rows - 1) * (unsigned)ld + DH) * 2u);
#pragma unroll
    for (int u = 0; u < Few<DH>::LOADS; ++u) buffer_to_lds(tile + 1024u * u, off[u], buf);
  }
};
// Lane L's 4 bytes at p land in LDS at lds + 4 L.
__device__ __forceinline__ void float_to_lds(unsigned lds, const float* p) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds), "v"(p) : "memory");
}

// A maximum in units of the exponent, rounded once: what a sum is scaled by cancels exactly where it is scaled again, between tiles, in
// the merge and in lse, which a product fused into those differences would not (scores of deviation 6, 2048 rows: lse 6.7e-8 off,
// as the 128-row blocks' is 5.5e-8).
__device__ __forceinline__ float exponent_of(float m, float c) {
#pragma clang fp contract(off)
  return m * c;
}

// c += rows of the tile times b over the head dimension.
template <int DH>
__device__ __forceinline__ f32x16 dot_tile(const char* tile, const bf16x8 (&b)[DH / 16], f32x16 c, int lane) {
#pragma unroll
  for (int kk = 0; kk < DH / 16; ++kk)
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_row_fragment<DH>(tile, lane & 31, 2 * kk + (lane >> 5)), b[kk], c, 0, 0, 0);
  return c;
}
// acc[d] += tile^T w over the tile's 32 rows.
template <int DH, bool EDGE>
__device__ __forceinline__ void accumulate_tile(f32x16 (&acc)[DH / 32], const char* tile, const f32x16& w, int lane) {
#pragma unroll
  for (int st = 0; st < 2; ++st) {
    const Weights<EDGE> terms = weights_of<EDGE>(w, 8 * st);
#pragma unroll
    for (int d = 0; d < DH / 32; ++d)
      acc[d] = multiply<EDGE>(read_tr_fragment<DH>(tile, 16 * st, 32 * d, lane), terms, acc[d]);
  }
}
template <int DH>
__device__ __forceinline__ void load_row(bf16x8 (&f)[DH / 16], const bf16* row, int half) {
#pragma unroll
  for (int kk = 0; kk < DH / 16; ++kk) f[kk] = *reinterpret_cast<const bf16x8*>(row + 16 * kk + 8 * half);
}
// A partial result of one wave in LDS: [register][lane].
template <int N>
__device__ __forceinline__ void put_partial(float* p, const f32x16 (&acc)[N], int lane) {
#pragma unroll
  for (int d = 0; d < N; ++d)
#pragma unroll
    for (int e = 0; e < 16; ++e) p[(d * 16 + e) * 64 + lane] = acc[d][e];
}
// The waves' rows to redo, left in LDS before the barrier: all of them, and this wave's share.
template <int W>
__device__ __forceinline__ uint32_t all_redo(const uint32_t* masks) {
  uint32_t m = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) m |= masks[w];
  return __builtin_amdgcn_readfirstlane(m);
}
template <int W>
__device__ __forceinline__ uint32_t share_of(uint32_t redo, int wave) {
  return redo & ((W == 8 ? 0x01010101u : 0x11111111u) << wave);
}
__device__ __forceinline__ void store4(bf16* p, const f32x4& v) {
  bf16x4 b;
#pragma unroll
  for (int r = 0; r < 4; ++r) b[r] = (bf16)v[r];
  *reinterpret_cast<bf16x4*>(p) = b;
}

}  // namespace

template <int DH, bool EDGE>
__global__ __launch_bounds__((64 * Few<DH, true>::W)) void attn_few_fwd_kernel(const bf16* __restrict__ qkv, bf16* __restrict__ o,
                                                                       float* __restrict__ lse, int s, int h, int hkv,
                                                                       int group, float scale) {
  using F = Few<DH, true>;
  constexpr int DT = DH / 32, W = F::W, PART = F::NS * F::STAGE / 4;
  extern __shared__ __align__(16) char smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  const int n_heads = h / DH, head = blockIdx.x % n_heads, q0 = ((int)gridDim.x - 1 - (int)blockIdx.x) / n_heads * kRows;
  const int q = q0 + (lane & 31), ld = h + 2 * hkv, n_tiles = q0 / kRows + 1;
  const float c = scale * kLog2e;
  const bf16* kbase = qkv + h + (head / group) * DH;
  const bf16* vbase = kbase + hkv;
  char* stages = smem + wave * F::NS * F::STAGE;
  const unsigned stages_lds = __builtin_amdgcn_readfirstlane((int)lds_byte(stages));
  const TileLoads<DH> loads(ld, lane);
  auto request = [&](int i, int t) {
    loads.request(stages_lds + i % F::NS * F::STAGE, kbase, ld, kRows * t, s);
    loads.request(stages_lds + i % F::NS * F::STAGE + F::TILE, vbase, ld, kRows * t, s);
  };
#pragma unroll
  for (int i = 0; i < F::NS; ++i)
    if (wave + i * W < n_tiles) request(i, wave + i * W);
  bf16x8 qf[DH / 16];
  load_row<DH>(qf, qkv + (size_t)min(q, s - 1) * ld + head * DH, half);  // (rows past the end: computed, not stored)
  f32x16 acc[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d) acc[d] = zero16();
  float m_run = -INFINITY, mc_run = -INFINITY, l_run = 0.f;
  for (int t = wave, i = 0; t < n_tiles; t += W, ++i) {
    const bool more = t + W < n_tiles;
    if (F::NS == 1) wait_loads<F::LOADS>();  // K is there, V may be on its way
    else if (more) wait_loads<2 * F::LOADS>();
    else wait_loads<0>();
    const char* ktile = stages + i % F::NS * F::STAGE;
    f32x16 p = dot_tile<DH>(ktile, qf, zero16(), lane);
    if (F::NS == 1 && more) {
      wait_lds_reads();
      loads.request(stages_lds, kbase, ld, kRows * (t + W), s);
    }
    if (t == n_tiles - 1) {  // the tile of the diagonal; keys past s lie beyond it for every row there is
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (kRows * t + 8 * (e >> 2) + 4 * half + (e & 3) > q) p[e] = -INFINITY;
    }
    float mx = m_run;
#pragma unroll
    for (int e = 0; e < 16; ++e) mx = fmaxf(mx, p[e]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mc_new = exponent_of(mx, c), mc = mx == -INFINITY ? 0.f : mc_new;  // scores that are all -inf add nothing, instead of inf - inf
    const float alpha = fast_exp2(mc_run - mc);
    float sum = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      p[e] = fast_exp2(fmaf(p[e], c, -mc));
      sum += p[e];
    }
    m_run = mx;
    mc_run = mc_new;
    l_run = l_run * alpha + sum;
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[d][e] *= alpha;
    if (F::NS == 1) {
      if (more) wait_loads<F::LOADS>();
      else wait_loads<0>();
    }
    accumulate_tile<DH, EDGE>(acc, ktile + F::TILE, p, lane);
    if (F::NS == 1 && more) {
      wait_lds_reads();
      loads.request(stages_lds + F::TILE, vbase, ld, kRows * (t + W), s);
    } else if (t + F::NS * W < n_tiles) {
      wait_lds_reads();
      request(i, t + F::NS * W);
    }
  }
  float* part = reinterpret_cast<float*>(smem);
  put_partial<DT>(part + wave * PART, acc, lane);
  float* stat = reinterpret_cast<float*>(smem + F::AFTER);
  uint32_t* redo_of = reinterpret_cast<uint32_t*>(stat + 2 * W * 64);
  stat[wave * 64 + lane] = m_run;
  stat[(W + wave) * 64 + lane] = l_run + __shfl_xor(l_run, 32, 64);
  if constexpr (EDGE) {
    const uint32_t mine = rows_to_redo(not_finite<DT>(acc), s - q0);
    if (lane == 0) redo_of[wave] = mine;
  }
  __syncthreads();
  // Wave w finishes register groups w, w + W, ..: group g is columns 32 (g / 4) + 8 (g % 4) + 4 half .. of every lane's row.
  float m = stat[lane], f[W], l = 0.f;
#pragma unroll
  for (int w = 1; w < W; ++w) m = fmaxf(m, stat[w * 64 + lane]);  // wave 0 has seen key 0: finite
  const float mc = exponent_of(m, c);
#pragma unroll
  for (int w = 0; w < W; ++w) {
    f[w] = fast_exp2(exponent_of(stat[w * 64 + lane], c) - mc);
    l += stat[(W + w) * 64 + lane] * f[w];
  }
  if constexpr (EDGE) {
    const uint32_t redo = all_redo<W>(redo_of) & rows_to_redo(!is_nan(l), 32);
    if (redo) redo_forward_rows<bf16, DH>(share_of<W>(redo, wave), q0, qkv, o, lse, s, h, hkv, group, head, scale);
    if (q >= s || (redo >> (lane & 31) & 1)) return;
  }
  const float inv = 1.0f / l;
#pragma unroll
  for (int g = wave; g < 4 * DT; g += W) {
    f32x4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float x = 0.f;
#pragma unroll
      for (int w = 0; w < W; ++w) x += part[w * PART + (4 * g + r) * 64 + lane] * f[w];
      v[r] = x * inv;
    }
    store4(o + (size_t)q * h + head * DH + 8 * g + 4 * half, v);
  }
  if (wave == 0 && half == 0) {
    // by whichever constant is the more exact: 1 / 8, or c ln 2, whose two roundings all but cancel
    const float log_l = __logf(l), ln2 = 0.6931471805599453f;
    lse[(size_t)head * s + q] = DH == 64 ? m * scale + fmaf(fmaf(-m, c, mc), ln2, log_l) : fmaf(mc, ln2, log_l);
  }
}

// Block `at` of heads * tiles, heaviest first: 32 query rows of a head.
template <int DH, bool EDGE>
__device__ __forceinline__ void few_dq_block(char* smem, int at, const bf16* __restrict__ qkv, const bf16* __restrict__ d_o,
                                             const float* __restrict__ lse, const float* __restrict__ delta,
                                             bf16* __restrict__ dqkv, int s, int h, int hkv, int group, float scale) {
  using F = Few<DH>;
  constexpr int DT = DH / 32, W = F::W, PART = F::NS * F::STAGE / 4;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  const int n_heads = h / DH, head = at % n_heads, q0 = ((s - 1) / kRows - at / n_heads) * kRows, q = q0 + (lane & 31);
  const int ld = h + 2 * hkv, qc = min(q, s - 1), n_tiles = q0 / kRows + 1;
  const float c = scale * kLog2e;
  const bf16* kbase = qkv + h + (head / group) * DH;
  const bf16* vbase = kbase + hkv;
  char* stages = smem + wave * F::NS * F::STAGE;
  const unsigned stages_lds = __builtin_amdgcn_readfirstlane((int)lds_byte(stages));
  const TileLoads<DH> loads(ld, lane);
  auto request = [&](int i, int t) {
    loads.request(stages_lds + i % F::NS * F::STAGE, kbase, ld, kRows * t, s);
    loads.request(stages_lds + i % F::NS * F::STAGE + F::TILE, vbase, ld, kRows * t, s);
  };
#pragma unroll
  for (int i = 0; i < F::NS; ++i)
    if (wave + i * W < n_tiles) request(i, wave + i * W);
  bf16x8 qf[DH / 16], dof[DH / 16];
  load_row<DH>(qf, qkv + (size_t)qc * ld + head * DH, half);
  load_row<DH>(dof, d_o + (size_t)qc * h + head * DH, half);
  const float lse_q = lse[(size_t)head * s + qc] * kLog2e, delta_q = delta[(size_t)head * s + qc];
  f32x16 dq[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d) dq[d] = zero16();
  for (int t = wave, i = 0; t < n_tiles; t += W, ++i) {
    if (t + W < n_tiles) wait_loads<2 * F::LOADS>();
    else wait_loads<0>();
    const char* ktile = stages + i % F::NS * F::STAGE;
    f32x16 p = dot_tile<DH>(ktile, qf, zero16(), lane);
    f32x16 ds = dot_tile<DH>(ktile + F::TILE, dof, zero16(), lane);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      float pe = fast_exp2(p[e] * c - lse_q);
      if (t == n_tiles - 1 && kRows * t + 8 * (e >> 2) + 4 * half + (e & 3) > q) pe = 0.f;
      ds[e] = pe * (ds[e] - delta_q);
    }
    accumulate_tile<DH, EDGE>(dq, ktile, ds, lane);
    wait_lds_reads();
    if (t + F::NS * W < n_tiles) request(i, t + F::NS * W);
  }
  float* part = reinterpret_cast<float*>(smem);
  put_partial<DT>(part + wave * PART, dq, lane);
  uint32_t* redo_of = reinterpret_cast<uint32_t*>(smem + F::AFTER);
  if constexpr (EDGE) {
    const uint32_t mine = rows_to_redo(not_finite<DT>(dq) && !is_nan(lse_q + delta_q), s - q0);
    if (lane == 0) redo_of[wave] = mine;
  }
  __syncthreads();
  if constexpr (EDGE) {
    const uint32_t redo = all_redo<W>(redo_of);
    if (redo)
      redo_dq_rows<bf16, DH>(share_of<W>(redo, wave), q0, qkv, d_o, lse, delta, dqkv, s, h, hkv, group, head, scale);
    if (q >= s || (redo >> (lane & 31) & 1)) return;
  }
#pragma unroll
  for (int g = wave; g < 4 * DT; g += W) {
    f32x4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float x = 0.f;
#pragma unroll
      for (int w = 0; w < W; ++w) x += part[w * PART + (4 * g + r) * 64 + lane];
      v[r] = x * scale;
    }
    store4(dqkv + (size_t)q * ld + head * DH + 8 * g + 4 * half, v);
  }
}

// Block `at` of (heads / hpb) * tiles, heaviest first: 32 keys of the key/value head that query heads bx hpb .. read, whose
// query tiles its waves walk.  partials (may be null): where dK and dV go in fp32, columns bx DH of the two halves of
// [s, 2 DH heads / hpb].
template <int DH, bool EDGE>
__device__ __forceinline__ void few_dkv_block(char* smem, int at, const bf16* __restrict__ qkv, const bf16* __restrict__ d_o,
                                              const float* __restrict__ lse, const float* __restrict__ delta,
                                              bf16* __restrict__ dqkv, float* __restrict__ partials, int hpb, int s, int h,
                                              int hkv, int group, float scale) {
  using F = Few<DH>;
  constexpr int DT = DH / 32, W = F::W, PART = F::NS * F::STAGE / 4;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  const int n_x = h / DH / hpb, bx = at % n_x, first = at / n_x, key = first * kRows + (lane & 31);
  const int kv_head = bx * hpb / group, ld = h + 2 * hkv, last = s - 1, n_q = last / kRows + 1 - first, n_it = hpb * n_q;
  const float c = scale * kLog2e, from_lse = -1.0f / scale;
  char* stages = smem + wave * F::NS * F::STAGE;
  char* stats = smem + F::AFTER + wave * F::NS * 256;  // per stage lse and delta of the tile's 32 rows
  const unsigned stages_lds = __builtin_amdgcn_readfirstlane((int)lds_byte(stages));
  const unsigned stats_lds = __builtin_amdgcn_readfirstlane((int)lds_byte(stats));
  const TileLoads<DH> q_loads(ld, lane), do_loads(h, lane);
  const float* stat_of = half ? delta : lse;
  auto request = [&](int i, int it) {
    const int g = it / n_q, q0 = (first + it - g * n_q) * kRows, head = bx * hpb + g;
    q_loads.request(stages_lds + i % F::NS * F::STAGE, qkv + head * DH, ld, q0, s);
    do_loads.request(stages_lds + i % F::NS * F::STAGE + F::TILE, d_o + head * DH, h, q0, s);
    float_to_lds(stats_lds + i % F::NS * 256, stat_of + (size_t)head * s + min(q0 + (lane & 31), last));
  };
#pragma unroll
  for (int i = 0; i < F::NS; ++i)
    if (wave + i * W < n_it) request(i, wave + i * W);
  bf16x8 kf[DH / 16], vf[DH / 16];
  const bf16* krow = qkv + (size_t)min(key, last) * ld + h + kv_head * DH;  // (keys past the end: computed, not stored)
  load_row<DH>(kf, krow, half);
  load_row<DH>(vf, krow + hkv, half);
  f32x16 dk[DT], dv[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d) dk[d] = dv[d] = zero16();
  for (int it = wave, i = 0; it < n_it; it += W, ++i) {
    const int g = it / n_q, q0 = (first + it - g * n_q) * kRows;
    if (it + W < n_it) wait_loads<2 * F::LOADS + 1>();
    else wait_loads<0>();
    const char* qtile = stages + i % F::NS * F::STAGE;
    const float* stat = reinterpret_cast<const float*>(stats + i % F::NS * 256);
    f32x16 p, ds;  // the row statistics are the initial value: S - lse / scale and dP - delta
#pragma unroll
    for (int b = 0; b < 4; ++b) {  // register 4 b + r is query row 8 b + 4 half + r
      const f32x4 vl = *reinterpret_cast<const f32x4*>(stat + 8 * b + 4 * half);
      const f32x4 vd = *reinterpret_cast<const f32x4*>(stat + 32 + 8 * b + 4 * half);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p[4 * b + r] = vl[r] * from_lse;
        ds[4 * b + r] = -vd[r];
      }
    }
    p = dot_tile<DH>(qtile, kf, p, lane);
    ds = dot_tile<DH>(qtile + F::TILE, vf, ds, lane);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      p[e] = fast_exp2(p[e] * c);
      ds[e] *= p[e];
    }
    if (q0 == first * kRows || q0 + kRows > s) {  // the diagonal, or rows past the end
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int q = q0 + 8 * (e >> 2) + 4 * half + (e & 3);
        // dS is selected too: 0 times the dP of a row that is not finite is no 0
        if (q > last || key > q) p[e] = ds[e] = 0.f;
      }
    }
    accumulate_tile<DH, EDGE>(dv, qtile + F::TILE, p, lane);
    accumulate_tile<DH, EDGE>(dk, qtile, ds, lane);
    wait_lds_reads();
    if (it + F::NS * W < n_it) request(i, it + F::NS * W);
  }
  float* part = reinterpret_cast<float*>(smem);
  put_partial<DT>(part + wave * PART, dk, lane);
  put_partial<DT>(part + wave * PART + PART / 2, dv, lane);
  __syncthreads();
  if (key > last) return;
  bf16* out = dqkv + (size_t)key * ld + h + kv_head * DH + 4 * half;
  float* part_out = partials + (size_t)key * 2 * n_x * DH + bx * DH + 4 * half;
#pragma unroll
  for (int g = wave; g < 4 * DT; g += W) {
    f32x4 vk, vv;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float x = 0.f, y = 0.f;
#pragma unroll
      for (int w = 0; w < W; ++w) {
        x += part[w * PART + (4 * g + r) * 64 + lane];
        y += part[w * PART + PART / 2 + (4 * g + r) * 64 + lane];
      }
      vk[r] = x * scale;
      vv[r] = y;
    }
    if (partials) {
      *reinterpret_cast<f32x4*>(part_out + 8 * g) = vk;
      *reinterpret_cast<f32x4*>(part_out + n_x * DH + 8 * g) = vv;
    } else {
      store4(out + 8 * g, vk);
      store4(out + hkv + 8 * g, vv);
    }
  }
}

template <int DH, bool EDGE>
__global__ __launch_bounds__(64 * Few<DH>::W) void attn_few_bwd_kernel(const bf16* __restrict__ qkv,
                                                                       const bf16* __restrict__ d_o,
                                                                       const float* __restrict__ lse,
                                                                       const float* __restrict__ delta,
                                                                       bf16* __restrict__ dqkv,
                                                                       float* __restrict__ partials, int hpb, int s, int h,
                                                                       int hkv, int group, float scale, int dkv_blocks) {
  extern __shared__ __align__(16) char smem[];
  if ((int)blockIdx.x < dkv_blocks)
    few_dkv_block<DH, EDGE>(smem, blockIdx.x, qkv, d_o, lse, delta, dqkv, partials, hpb, s, h, hkv, group, scale);
  else
    few_dq_block<DH, EDGE>(smem, blockIdx.x - dkv_blocks, qkv, d_o, lse, delta, dqkv, s, h, hkv, group, scale);
}

// ---- host side -------------------------------------------------------------------------------------------------
// Which of two launches is the faster hangs on their blocks: as long as the blocks of 32 rows find a place within a round or two,
// their chains, a quarter as long, win, and the longer the sequence the more rounds that outweighs; beyond, the 128-row blocks' use
// of a tile for four times the rows does.  Lines drawn over 4800 calls of 4000 shapes (1 to 300 heads, groups of 1, 2 and 4, 1 to 15000
// rows, at 0.25 to 1.15 times the line), both kinds of blocks in turn: none of these took over 3 % longer.  128-row / 32-row blocks, us,
// forward and backward:
//   8 heads of 64, 512 rows        8.9 /   5.7   16.9 /   9.9      16 heads of 128, 100 rows           9.8 /   5.6   18.0 /  10.9
//   8 heads of 64, 1024 rows      12.5 /   7.9   25.4 /  16.2      4 heads of 128, 2048 rows          27.4 /  18.3   64.6 /  38.6
//   10 heads of 64 over 2, 777    15.6 /   8.3    137 /  35.9      16 heads of 128, 1024 rows (not)   17.7 /  16.5   41.2 /  46.1
//   32 heads of 64, 512 (not)      9.2 /   8.5   17.8 /  22.7      16 heads of 128, 2048 rows (not)   30.1 /  42.2   83.2 /   130
static bool offsets_fit(int h, int n_heads, int n_kv_heads) {  // a lane's offset in a tile of 32 rows
  return ((int64_t)h + 2 * (int64_t)n_kv_heads * (h / n_heads)) * (2 * kRows) < (int64_t)1 << 32;
}
constexpr int kFewHeads = 150;  // tiles from which on the caps leave a handful of heads, whose chains decide
bool attention_few_forward_is_faster(int s, int h, int n_heads, int n_kv_heads) {
  const int64_t tiles = ceil_div(s, kRows), blocks = n_heads * tiles;
  const bool whole = s % 128 == 0;
  // 32 x 544 / 14 x 518 / 72 x 936 / 93 x 1023 blocks (tiles x blocks) of heads of 64 took 5 / 6 / 4 / 3 % longer, 112 x 1008 of 128 4 %
  const bool few_heads = tiles > kFewHeads;
  const int64_t line = h / n_heads == 64
                           ? (whole ? std::min<int64_t>(768, 412 + 4 * tiles) : std::min<int64_t>(few_heads ? 1024 : 928, 408 + 7 * tiles))
                           : (whole ? std::min<int64_t>(768, 352 + 2 * tiles) : std::min<int64_t>(few_heads ? 1024 : 864, 416 + 6 * tiles));
  return blocks <= line && offsets_fit(h, n_heads, n_kv_heads);
}
// A dK/dV block's chain grows with the query heads it walks: without partial results 8 heads of 128 over 1 at 1000 rows 118 /
// 146 us, 16 heads of 64 over 2 at 847 rows 65 / 56, 16 heads of 128 over 1 at 30 rows 25 / 18.  But so does a 128-row block's, and groups
// win by a fifth and more up to their lines.  Without groups the lines are lower: one round of 256 blocks where 128-row blocks
// waste few rows (96 heads of 64 at 66 rows 11.2 / 13.3, 36 at 256 rows 13.2 / 14.4, 25 at 384 rows 15.6 / 16.6), and caps (10 heads of 64
// at 3250 rows 115 / 128, 9 at 2048 rows 44.1 / 46.6, 11 heads of 128 at 2565 rows 168 / 186, 9 at 1792 rows 63.9 / 68.6).
bool attention_few_backward_is_faster(int s, int h, int n_heads, int n_kv_heads, int hpb) {
  const int64_t tiles = ceil_div(s, kRows), blocks = n_heads * tiles;
  const bool whole = s % 128 == 0;
  const int waves = h / n_heads == 64 ? Few<64>::W : Few<128>::W;
  int64_t line = h / n_heads == 64 ? (whole ? std::min<int64_t>(640, 256 + 5 * tiles) : std::min<int64_t>(1024, 288 + 8 * tiles))
                                   : (whole ? std::min<int64_t>(512, 224 + 5 * tiles) : std::min<int64_t>(896, 288 + 8 * tiles));
  if (hpb == 1) {
    const bool few_heads = tiles > kFewHeads;
    if (!whole) {
      const int64_t cap = h / n_heads == 64 ? (few_heads ? 1024 : 768) : (few_heads ? 896 : 720);
      line = tiles == 3 || tiles == 4 ? 256 : std::min(line, cap);
    } else if (h / n_heads == 64) {
      line = std::min(line, std::min<int64_t>(few_heads ? 640 : 560, std::max<int64_t>(256, 160 + 8 * tiles)));
    } else {
      line = std::min<int64_t>(few_heads ? 512 : 448, 224 + 4 * tiles);
    }
  }
  return blocks <= line && (hpb <= (whole ? waves / 2 : waves) || hpb * tiles <= 24) && offsets_fit(h, n_heads, n_kv_heads);
}

template <int DH, bool EDGE>
static bool few_forward(const bf16* qkv, bf16* o, float* lse, int s, int h, int n_heads, int n_kv_heads, hipStream_t stream) {
  using F = Few<DH, true>;
  constexpr int smem = F::AFTER + 2 * F::W * 256 + F::W * 4;
  static LdsLimit lds;
  if (!lds.allow(attn_few_fwd_kernel<DH, EDGE>, smem)) return false;
  attn_few_fwd_kernel<DH, EDGE><<<n_heads * ceil_div(s, kRows), 64 * F::W, smem, stream>>>(
      qkv, o, lse, s, h, n_kv_heads * DH, n_heads / n_kv_heads, 1.0f / sqrtf((float)DH));
  return launch_ok("attn_few_fwd_kernel");
}
bool attention_few_forward(const bf16* qkv, bf16* o, float* lse, int s, int h, int n_heads, int n_kv_heads,
                           hipStream_t stream) {
  auto launch = s % 128 == 0 ? (h / n_heads == 128 ? few_forward<128, false> : few_forward<64, false>)
                             : (h / n_heads == 128 ? few_forward<128, true> : few_forward<64, true>);
  return launch(qkv, o, lse, s, h, n_heads, n_kv_heads, stream);
}

template <int DH, bool EDGE>
static bool few_backward(const bf16* qkv, const float* lse, const float* delta, const bf16* d_o, bf16* dqkv, float* partials,
                         int hpb, int s, int h, int n_heads, int n_kv_heads, hipStream_t stream) {
  constexpr int smem = Few<DH>::AFTER + Few<DH>::W * Few<DH>::NS * 256;
  static LdsLimit lds;
  if (!lds.allow(attn_few_bwd_kernel<DH, EDGE>, smem)) return false;
  const int tiles = ceil_div(s, kRows), dkv_blocks = n_heads / hpb * tiles;
  attn_few_bwd_kernel<DH, EDGE><<<dkv_blocks + n_heads * tiles, 64 * Few<DH>::W, smem, stream>>>(
      qkv, d_o, lse, delta, dqkv, partials, hpb, s, h, n_kv_heads * DH, n_heads / n_kv_heads, 1.0f / sqrtf((float)DH),
      dkv_blocks);
  return launch_ok("attn_few_bwd_kernel");
}
bool attention_few_backward(const bf16* qkv, const float* lse, const float* delta, const bf16* d_o, bf16* dqkv,
                            float* partials, int hpb, int s, int h, int n_heads, int n_kv_heads, hipStream_t stream) {
  auto launch = s % 128 == 0 ? (h / n_heads == 128 ? few_backward<128, false> : few_backward<64, false>)
                             : (h / n_heads == 128 ? few_backward<128, true> : few_backward<64, true>);
  return launch(qkv, lse, delta, d_o, dqkv, partials, hpb, s, h, n_heads, n_kv_heads, stream);
}

}  // namespace po
