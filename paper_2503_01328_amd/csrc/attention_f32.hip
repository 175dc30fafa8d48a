// fp32 causal attention on the matrix cores (v_mfma_f32_32x32x2_f32: full fp32 products and sums), forward and
// backward, any sequence length, head sizes 32, 64, 96 and 128.
//
// An fp32 MFMA takes 64 cycles for two operand registers, so nothing has to be staged through LDS to feed it: every
// wave works on its own, operands straight from global memory (they stay in L2: a head's K and V) into registers, no
// barrier in the loops.  What counts is that every SIMD has a wave and that no chain is long: a block owns only 32
// rows (query rows in forward and dQ, keys in dK/dV) and its four waves split the tiles of 32 keys (query rows) those
// meet, tile t to wave t % 4; the four partial results are added in wave order through LDS at the end (deterministic,
// no atomics).  Heaviest blocks of the causal triangle first.
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
// s = 1024, 16 heads of 64: forward 38 us (2 s^2 h: 56 of 157 TFLOP/s), dK/dV 87 us, dQ 54 us; the vector kernels of
// attention_generic.hip take 625, 3076 and 769 us.  s = 128, 4 heads: 7.6, 12.8 and 9.1 us (44, 55 and 28 us), there
// bound by the chain of one tile: two loads, 64 to 128 dependent MFMAs, the sum over the waves.
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
template <int DH>
__device__ __forceinline__ f32x16 dot_tile(const f32x4 (&a)[DH / 8], const f32x4 (&b)[DH / 8]) {
  f32x16 c = zero16();
#pragma unroll
  for (int kk = 0; kk < DH / 8; ++kk)
#pragma unroll
    for (int j = 0; j < 4; ++j) c = mfma(a[kk][j], b[kk][j], c);
  return c;
}
// acc[d] += M^T w over the 32 rows from row0 on: first operand rows of M (clamped to the last), second w.
template <int DH>
__device__ __forceinline__ void accumulate_rows(f32x16 (&acc)[DH / 32], const float* m, int ld, int row0, int last,
                                                const f32x16& w, int lane) {
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const float* row = m + (size_t)min(row0 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3), last) * ld + (lane & 31);
#pragma unroll
    for (int d = 0; d < DH / 32; ++d) acc[d] = mfma(row[32 * d], w[e], acc[d]);
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

}  // namespace

template <int DH>
__global__ __launch_bounds__(256, 2) void attn_f32_fwd_kernel(const float* __restrict__ qkv, float* __restrict__ o,
                                                              float* __restrict__ lse, int s, int h, int hkv, int group,
                                                              float scale) {
  constexpr int DT = DH / 32, PART = DT * 16 * 64;
  extern __shared__ __align__(16) float lds[];  // four partial outputs, then their maxima and row sums, rows to redo
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  const int head = blockIdx.x, q0 = (int)(gridDim.y - 1 - blockIdx.y) * 32, q = q0 + (lane & 31);
  const int ld = h + 2 * hkv, last = s - 1;
  const float* kbase = qkv + h + (head / group) * DH;
  const float* vbase = kbase + hkv;
  f32x4 qf[DH / 8];
  load_pieces<DH>(qf, qkv + (size_t)min(q, last) * ld + head * DH, half);
  f32x16 acc[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d) acc[d] = zero16();
  float m_run = -INFINITY, l_run = 0.f;
  const int n_tiles = min(q0 + 31, last) / 32 + 1;
  for (int t = wave; t < n_tiles; t += 4) {
    f32x4 kf[DH / 8];
    load_pieces<DH>(kf, kbase + (size_t)min(32 * t + (lane & 31), last) * ld, half);
    f32x16 p = dot_tile<DH>(kf, qf);
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
    accumulate_rows<DH>(acc, vbase, ld, 32 * t, last, p, lane);
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

template <int DH>
__global__ __launch_bounds__(256, DH > 64 ? 1 : 2) void attn_f32_bwd_dq_kernel(
    const float* __restrict__ qkv, const float* __restrict__ d_o, const float* __restrict__ lse,
    const float* __restrict__ delta, float* __restrict__ dqkv, int s, int h, int hkv, int group, float scale) {
  constexpr int DT = DH / 32, PART = DT * 16 * 64;
  extern __shared__ __align__(16) float lds[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  const int head = blockIdx.x, q0 = (int)(gridDim.y - 1 - blockIdx.y) * 32, q = q0 + (lane & 31);
  const int ld = h + 2 * hkv, last = s - 1, qc = min(q, last);
  const float* kbase = qkv + h + (head / group) * DH;
  const float* vbase = kbase + hkv;
  f32x4 qf[DH / 8], dof[DH / 8];
  load_pieces<DH>(qf, qkv + (size_t)qc * ld + head * DH, half);
  load_pieces<DH>(dof, d_o + (size_t)qc * h + head * DH, half);
  const float lse_q = lse[(size_t)head * s + qc], delta_q = delta[(size_t)head * s + qc];
  f32x16 dq[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d) dq[d] = zero16();
  const int n_tiles = min(q0 + 31, last) / 32 + 1;
  for (int t = wave; t < n_tiles; t += 4) {
    const size_t row = (size_t)min(32 * t + (lane & 31), last) * ld;
    f32x4 kf[DH / 8];
    load_pieces<DH>(kf, kbase + row, half);
    f32x16 p = dot_tile<DH>(kf, qf);
    load_pieces<DH>(kf, vbase + row, half);
    f32x16 ds = dot_tile<DH>(kf, dof);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      float pe = __builtin_amdgcn_exp2f(fmaf(p[e], scale, -lse_q) * kLog2e);
      if (t == n_tiles - 1 && 32 * t + 8 * (e >> 2) + 4 * half + (e & 3) > q) pe = 0.f;
      ds[e] = pe * (ds[e] - delta_q);
    }
    accumulate_rows<DH>(dq, kbase, ld, 32 * t, last, ds, lane);
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

// Block: 32 keys of one key/value head; its waves walk the query tiles of every query head that reads it.
template <int DH>
__global__ __launch_bounds__(256, 1) void attn_f32_bwd_dkv_kernel(
    const float* __restrict__ qkv, const float* __restrict__ d_o, const float* __restrict__ lse,
    const float* __restrict__ delta, float* __restrict__ dqkv, int s, int h, int hkv, int group, float scale) {
  constexpr int DT = DH / 32, PART = DT * 16 * 64;
  extern __shared__ __align__(16) float lds[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  const int kv_head = blockIdx.x, first = blockIdx.y, key = first * 32 + (lane & 31);
  const int ld = h + 2 * hkv, last = s - 1;
  f32x4 kf[DH / 8], vf[DH / 8];
  const float* krow = qkv + (size_t)min(key, last) * ld + h + kv_head * DH;
  load_pieces<DH>(kf, krow, half);
  load_pieces<DH>(vf, krow + hkv, half);
  f32x16 dk[DT], dv[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d) dk[d] = dv[d] = zero16();
  const int n_q = last / 32 + 1 - first, n_it = group * n_q;
  for (int it = wave; it < n_it; it += 4) {
    const int g = it / n_q, q0 = (first + it - g * n_q) * 32, head = kv_head * group + g;
    const float* qbase = qkv + head * DH;
    const float* dobase = d_o + head * DH;
    const int row = min(q0 + (lane & 31), last);
    f32x4 a[DH / 8];
    load_pieces<DH>(a, qbase + (size_t)row * ld, half);
    f32x16 p = dot_tile<DH>(a, kf);
    load_pieces<DH>(a, dobase + (size_t)row * h, half);
    f32x16 ds = dot_tile<DH>(a, vf);
    const float* lse_h = lse + (size_t)head * s;
    const float* delta_h = delta + (size_t)head * s;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int qc = min(q0 + 8 * (e >> 2) + 4 * half + (e & 3), last);
      p[e] = __builtin_amdgcn_exp2f(fmaf(p[e], scale, -lse_h[qc]) * kLog2e);
      ds[e] = p[e] * (ds[e] - delta_h[qc]);
    }
    if (q0 == first * 32 || q0 + 31 > last) {  // the diagonal, or rows past the end
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int q = q0 + 8 * (e >> 2) + 4 * half + (e & 3);
        // dS is selected too: 0 times the dP of a row that is not finite is no 0
        if (q > last || key > q) p[e] = ds[e] = 0.f;
      }
    }
    accumulate_rows<DH>(dv, dobase, h, q0, last, p, lane);
    accumulate_rows<DH>(dk, qbase, ld, q0, last, ds, lane);
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

// ---- host side -------------------------------------------------------------------------------------------------
bool attention_f32_supported(const void* qkv, const void* o, int s, int h, int n_heads, int n_kv_heads) {
  if (s <= 0 || h <= 0 || n_heads <= 0 || h % n_heads != 0 || n_kv_heads <= 0 || n_heads % n_kv_heads != 0) return false;
  if (s > 32 * kMaxGridY) return false;
  const int dh = h / n_heads;
  return (dh == 32 || dh == 64 || dh == 96 || dh == 128) && ((uintptr_t)qkv | (uintptr_t)o) % 16 == 0;
}

template <int DH>
static bool forward_f32(const float* qkv, float* o, float* lse, int s, int h, int n_heads, int n_kv_heads,
                        hipStream_t stream) {
  constexpr int smem = (4 * DH * 32 + 8 * 64 + 4) * 4;
  static LdsLimit lds;
  if (!lds.allow(attn_f32_fwd_kernel<DH>, smem)) return false;
  attn_f32_fwd_kernel<DH><<<dim3(n_heads, ceil_div(s, 32)), 256, smem, stream>>>(
      qkv, o, lse, s, h, n_kv_heads * DH, n_heads / n_kv_heads, 1.0f / sqrtf((float)DH));
  return launch_ok("attn_f32_fwd_kernel");
}

template <int DH>
static bool backward_f32(const float* qkv, const float* lse, const float* delta, const float* d_o, float* dqkv, int s,
                         int h, int n_heads, int n_kv_heads, hipStream_t stream) {
  constexpr int smem_part = 4 * DH * 32 * 4, smem_q = smem_part + 16, smem_kv = 2 * smem_part;
  static LdsLimit lds_q, lds_kv;
  if (!lds_q.allow(attn_f32_bwd_dq_kernel<DH>, smem_q) || !lds_kv.allow(attn_f32_bwd_dkv_kernel<DH>, smem_kv)) return false;
  const int hkv = n_kv_heads * DH, group = n_heads / n_kv_heads;
  const float scale = 1.0f / sqrtf((float)DH);
  attn_f32_bwd_dkv_kernel<DH><<<dim3(n_kv_heads, ceil_div(s, 32)), 256, smem_kv, stream>>>(qkv, d_o, lse, delta, dqkv, s,
                                                                                          h, hkv, group, scale);
  attn_f32_bwd_dq_kernel<DH><<<dim3(n_heads, ceil_div(s, 32)), 256, smem_q, stream>>>(qkv, d_o, lse, delta, dqkv, s, h,
                                                                                      hkv, group, scale);
  return launch_ok("attn_f32_bwd kernels");
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

}  // namespace po
