// Causal attention on the vector ALU for any dtype, sequence length and head
// size up to 256: what force_generic asks for and the home of shapes the
// matrix-core kernels do not take.  One wave owns one (head, row): lanes split the keys of a
// 64-wide chunk for the scores (online softmax, running max and sum), then
// split the head dimension for the weighted sums, the per-key weights being
// broadcast with shuffles.  Backward is split into a dQ kernel (wave per query
// row) and a dK/dV kernel (wave per key row), each summing in a fixed order, so
// there are no atomics and results are reproducible.
//
// Grouped-query attention: the qkv matrix is [s, h + 2 hkv] (query block, key block, value block) with
// hkv = n_kv_heads * dh; query head t reads key/value head t / group, group = n_heads / n_kv_heads.  The dK/dV
// kernel runs per key/value head and walks its group's query heads in order.
#include "attention_rows.h"
#include "kernels.h"

namespace po {

constexpr int kMaxHeadDim = 256;
constexpr int kDimSlots = kMaxHeadDim / kWave;  // head-dim elements per lane

template <typename T>
__global__ __launch_bounds__(256) void attn_fwd_generic_kernel(const T* __restrict__ qkv, T* __restrict__ o,
                                                               float* __restrict__ lse, int s, int h, int dh,
                                                               int hkv, int group, float scale) {
  __shared__ float qs[4][kMaxHeadDim];
  int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int head = blockIdx.y;
  int i = blockIdx.x * 4 + wave;
  bool active = i < s;
  int ld = h + 2 * hkv;
  const T* kbase = qkv + h + (head / group) * dh;
  const T* vbase = qkv + h + hkv + (head / group) * dh;
  if (active)
    for (int e = lane; e < dh; e += kWave) qs[wave][e] = to_f32(qkv[(size_t)i * ld + head * dh + e]) * scale;
  __syncthreads();
  if (!active) return;
  attention_forward_row<T, kDimSlots, 1>([&](int e) { return qs[wave][e]; }, kbase, vbase, ld, i, dh, lane,
                                      o + (size_t)i * h + head * dh, lse + (size_t)head * s + i);
}

// delta[head][i] = sum_e dO[i, head, e] * O[i, head, e]
template <typename T>
__global__ __launch_bounds__(256) void attn_delta_kernel(const T* __restrict__ o, const T* __restrict__ d_o,
                                                         float* __restrict__ delta, int s, int h, int dh) {
  int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int head = blockIdx.y;
  int i = blockIdx.x * 4 + wave;
  if (i >= s) return;
  float d = 0.f;
  for (int e = lane; e < dh; e += kWave) {
    size_t idx = (size_t)i * h + head * dh + e;
    d = fmaf(to_f32(o[idx]), to_f32(d_o[idx]), d);
  }
  d = wave_sum(d);
  if (lane == 0) delta[(size_t)head * s + i] = d;
}

template <typename T>
__global__ __launch_bounds__(256) void attn_bwd_dq_generic_kernel(const T* __restrict__ qkv,
                                                                  const float* __restrict__ lse,
                                                                  const float* __restrict__ delta,
                                                                  const T* __restrict__ d_o, T* __restrict__ dqkv,
                                                                  int s, int h, int dh, int hkv, int group,
                                                                  float scale) {
  __shared__ float qs[4][kMaxHeadDim];
  __shared__ float dos[4][kMaxHeadDim];
  int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int head = blockIdx.y;
  int i = blockIdx.x * 4 + wave;
  bool active = i < s;
  int ld = h + 2 * hkv;
  const T* kbase = qkv + h + (head / group) * dh;
  const T* vbase = qkv + h + hkv + (head / group) * dh;
  if (active)
    for (int e = lane; e < dh; e += kWave) {
      qs[wave][e] = to_f32(qkv[(size_t)i * ld + head * dh + e]) * scale;
      dos[wave][e] = to_f32(d_o[(size_t)i * h + head * dh + e]);
    }
  __syncthreads();
  if (!active) return;
  attention_dq_row<T, kDimSlots, 1>([&](int e) { return qs[wave][e]; }, [&](int e) { return dos[wave][e]; }, kbase, vbase, ld,
                                 lse[(size_t)head * s + i], delta[(size_t)head * s + i], i, dh, lane, scale,
                                 dqkv + (size_t)i * ld + head * dh);
}

template <typename T>
__global__ __launch_bounds__(256) void attn_bwd_dkv_generic_kernel(const T* __restrict__ qkv,
                                                                   const float* __restrict__ lse,
                                                                   const float* __restrict__ delta,
                                                                   const T* __restrict__ d_o, T* __restrict__ dqkv,
                                                                   int s, int h, int dh, int hkv, int group,
                                                                   float scale) {
  __shared__ float ks[4][kMaxHeadDim];
  __shared__ float vs[4][kMaxHeadDim];
  int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int kv_head = blockIdx.y;
  int j = blockIdx.x * 4 + wave;
  bool active = j < s;
  int ld = h + 2 * hkv;
  if (active)
    for (int e = lane; e < dh; e += kWave) {
      ks[wave][e] = to_f32(qkv[(size_t)j * ld + h + kv_head * dh + e]) * scale;
      vs[wave][e] = to_f32(qkv[(size_t)j * ld + h + hkv + kv_head * dh + e]);
    }
  __syncthreads();
  if (!active) return;
  float dk[kDimSlots], dv[kDimSlots];
#pragma unroll
  for (int r = 0; r < kDimSlots; ++r) dk[r] = dv[r] = 0.f;
  for (int g = 0; g < group; ++g) {  // the query heads that read this key/value head, in head order
    int head = kv_head * group + g;
    const T* qbase = qkv + head * dh;
    const T* dobase = d_o + head * dh;
    for (int i0 = j - (j % kWave); i0 < s; i0 += kWave) {
      int i = i0 + lane;
      float p = 0.f, ds = 0.f;
      if (i >= j && i < s) {
        const T* qr = qbase + (size_t)i * ld;
        const T* dor = dobase + (size_t)i * h;
        float sc = 0.f, dp = 0.f;
        for (int e = 0; e < dh; ++e) {
          sc = fmaf(ks[wave][e], to_f32(qr[e]), sc);
          dp = fmaf(vs[wave][e], to_f32(dor[e]), dp);
        }
        p = __expf(sc - lse[(size_t)head * s + i]);
        ds = p * (dp - delta[(size_t)head * s + i]);
      }
      int ni = min(kWave, s - i0);
      for (int ii = 0; ii < ni; ++ii) {
        float pi = __shfl(p, ii, kWave), dsi = __shfl(ds, ii, kWave);
        const T* qr = qbase + (size_t)(i0 + ii) * ld;
        const T* dor = dobase + (size_t)(i0 + ii) * h;
#pragma unroll
        for (int r = 0; r < kDimSlots; ++r) {
          int e = lane + kWave * r;
          if (e < dh) {
            dv[r] = fmaf(pi, to_f32(dor[e]), dv[r]);
            dk[r] = fmaf(dsi, to_f32(qr[e]), dk[r]);
          }
        }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < kDimSlots; ++r) {
    int e = lane + kWave * r;
    if (e < dh) {
      dqkv[(size_t)j * ld + h + kv_head * dh + e] = from_f32<T>(dk[r] * scale);
      dqkv[(size_t)j * ld + h + hkv + kv_head * dh + e] = from_f32<T>(dv[r]);
    }
  }
}

static bool check_attention_shape(const char* what, int s, int h, int n_heads, int n_kv_heads) {
  if (s <= 0 || h <= 0 || n_heads <= 0 || h % n_heads != 0 || h / n_heads > kMaxHeadDim || n_kv_heads <= 0 ||
      n_heads % n_kv_heads != 0) {
    set_error("%s: s=%d h=%d heads=%d kv_heads=%d (head size must divide h and be <= %d, kv_heads must divide heads)",
              what, s, h, n_heads, n_kv_heads, kMaxHeadDim);
    return false;
  }
  return true;
}

bool attention_forward_generic(int dtype, const void* qkv, void* o, float* lse, int s, int h, int n_heads,
                               int n_kv_heads, hipStream_t stream) {
  if (!check_attention_shape("attention_forward", s, h, n_heads, n_kv_heads)) return false;
  int dh = h / n_heads, hkv = n_kv_heads * dh, group = n_heads / n_kv_heads;
  float scale = 1.0f / sqrtf((float)dh);
  dim3 grid(ceil_div(s, 4), n_heads);
  if (dtype == kF32)
    attn_fwd_generic_kernel<float><<<grid, 256, 0, stream>>>((const float*)qkv, (float*)o, lse, s, h, dh, hkv, group,
                                                             scale);
  else
    attn_fwd_generic_kernel<bf16><<<grid, 256, 0, stream>>>((const bf16*)qkv, (bf16*)o, lse, s, h, dh, hkv, group,
                                                            scale);
  return launch_ok("attn_fwd_generic_kernel");
}

bool attention_backward_generic(int dtype, const void* qkv, const void* o, const float* lse, const void* d_o,
                                void* dqkv, float* delta, int s, int h, int n_heads, int n_kv_heads,
                                hipStream_t stream) {
  if (!check_attention_shape("attention_backward", s, h, n_heads, n_kv_heads)) return false;
  int dh = h / n_heads, hkv = n_kv_heads * dh, group = n_heads / n_kv_heads;
  float scale = 1.0f / sqrtf((float)dh);
  dim3 grid(ceil_div(s, 4), n_heads), grid_kv(ceil_div(s, 4), n_kv_heads);
  if (dtype == kF32) {
    attn_delta_kernel<float><<<grid, 256, 0, stream>>>((const float*)o, (const float*)d_o, delta, s, h, dh);
    attn_bwd_dq_generic_kernel<float><<<grid, 256, 0, stream>>>((const float*)qkv, lse, delta, (const float*)d_o,
                                                                (float*)dqkv, s, h, dh, hkv, group, scale);
    attn_bwd_dkv_generic_kernel<float><<<grid_kv, 256, 0, stream>>>((const float*)qkv, lse, delta,
                                                                    (const float*)d_o, (float*)dqkv, s, h, dh, hkv,
                                                                    group, scale);
  } else {
    attn_delta_kernel<bf16><<<grid, 256, 0, stream>>>((const bf16*)o, (const bf16*)d_o, delta, s, h, dh);
    attn_bwd_dq_generic_kernel<bf16><<<grid, 256, 0, stream>>>((const bf16*)qkv, lse, delta, (const bf16*)d_o,
                                                               (bf16*)dqkv, s, h, dh, hkv, group, scale);
    attn_bwd_dkv_generic_kernel<bf16><<<grid_kv, 256, 0, stream>>>((const bf16*)qkv, lse, delta, (const bf16*)d_o,
                                                                   (bf16*)dqkv, s, h, dh, hkv, group, scale);
  }
  return launch_ok("attention backward kernels");
}

// Whether a bf16 call goes to the matrix-core kernels, which load 16 bytes at a time: sequences of whole tiles always
// do (they refuse other alignments), the others where every tensor is aligned so.
static bool vectors_or_refused(int s, uintptr_t addresses) { return s % 128 == 0 || addresses % 16 == 0; }

bool attention_forward(int dtype, const void* qkv, void* o, float* lse, int s, int h, int n_heads, int n_kv_heads,
                       bool force_generic, hipStream_t stream) {
  // Vector / matrix cores in us, 16 heads: of 64 at 16, 43 and 51 rows 6.6 / 4.0, 11.3 / 4.1 and 12.6 / 4.1, of 128 at 64
  // rows 21.7 / 5.0.  The line was drawn when the matrix-core kernel took 10.6 and 17.5 us at any
  // of these and has not been moved since.  The backward has none (8 rows: 15.5 / 7.1 and 24.6 / 9.5).
  const int few = h == 64 * (int64_t)n_heads ? 43 : 51;
  if (dtype == kBF16 && !force_generic && s > few && attention_mfma_supported(s, h, n_heads, n_kv_heads) &&
      vectors_or_refused(s, (uintptr_t)qkv | (uintptr_t)o))
    return attention_forward_mfma(qkv, o, lse, s, h, n_heads, n_kv_heads, stream);
  // fp32, vector / matrix cores at few rows (8 heads), us: heads of 32 at 8 rows 5.3 / 4.8; of 64 at 8 and 14 rows 5.4 / 6.2 and
  // 6.3 / 6.2; of 96 at 8 and 14 rows 6.7 / 7.7 and 8.2 / 7.7; of 128 at 8, 16 and 19 rows 7.2 / 8.9, 9.3 / 8.9 and 9.9 / 8.9:
  // the chain of one tile against one key after the other.
  if (dtype == kF32 && !force_generic && 64 * (int64_t)s > 9 * (int64_t)(h / max(n_heads, 1)) &&
      attention_f32_supported(qkv, o, s, h, n_heads, n_kv_heads))
    return attention_forward_f32((const float*)qkv, (float*)o, lse, s, h, n_heads, n_kv_heads, stream);
  return attention_forward_generic(dtype, qkv, o, lse, s, h, n_heads, n_kv_heads, stream);
}

bool attention_backward(int dtype, const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv,
                        float* delta, void* partials, int s, int h, int n_heads, int n_kv_heads, bool force_generic,
                        hipStream_t stream) {
  if (dtype == kBF16 && !force_generic && attention_mfma_supported(s, h, n_heads, n_kv_heads) &&
      vectors_or_refused(s, (uintptr_t)qkv | (uintptr_t)o | (uintptr_t)d_o | (uintptr_t)dqkv))
    return attention_backward_mfma(qkv, o, lse, d_o, dqkv, delta, partials, s, h, n_heads, n_kv_heads, stream);
  // fp32 as in the forward: heads of 32 at 8 rows 12.0 / 8.2; of 64 at 12 and 14 rows 16.6 / 10.5 and 17.2 / 10.5; of 96 at 16
  // and 20 rows 23.6 / 14.3 and 26.8 / 14.4; of 128 at 20 and 26 rows 29.2 / 17.7 and 33.3 / 17.7 (the line was drawn when the
  // matrix-core kernels took 11.8 to 29 us and has not been moved since).
  if (dtype == kF32 && !force_generic && 64 * (int64_t)s > 12 * (int64_t)(h / max(n_heads, 1)) &&
      attention_f32_supported(qkv, d_o, s, h, n_heads, n_kv_heads) && (uintptr_t)dqkv % 16 == 0) {
    if ((uintptr_t)o % 16 != 0)
      attn_delta_kernel<float><<<dim3(ceil_div(s, 4), n_heads), 256, 0, stream>>>((const float*)o, (const float*)d_o, delta,
                                                                                 s, h, h / n_heads);
    else if (!attention_delta_f32((const float*)o, (const float*)d_o, delta, s, h, n_heads, stream))
      return false;
    return attention_backward_f32((const float*)qkv, lse, delta, (const float*)d_o, (float*)dqkv, s, h, n_heads,
                                  n_kv_heads, stream);
  }
  return attention_backward_generic(dtype, qkv, o, lse, d_o, dqkv, delta, s, h, n_heads, n_kv_heads, stream);
}

}  // namespace po
