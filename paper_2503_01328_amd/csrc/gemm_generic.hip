// Shape-agnostic GEMM on the vector ALU: the home of what the matrix-core kernels do not take (rows that are no whole
// 16-byte vectors, unaligned operands) and what force_generic asks for.  64x64 block tile,
// 16-deep k slices staged through LDS as fp32, each thread owns a 4x4 micro-tile.
// All bounds are checked, so any M, N, K >= 1 and any leading dimension works.
#include "column_sums.h"

namespace po {

template <typename T>
__global__ __launch_bounds__(256) void gemm_generic_kernel(int trans_a, int trans_b, int M, int N, int K,
                                                           const T* __restrict__ A, int lda,
                                                           const T* __restrict__ B, int ldb, Epilogue ep) {
  constexpr int BM = 64, BN = 64, BK = 16;
  __shared__ float As[BK][BM + 4];
  __shared__ float Bs[BK][BN + 4];
  int tid = threadIdx.x;
  int tx = tid & 15, ty = tid >> 4;  // micro-tile column / row index
  int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;

  for (int k0 = 0; k0 < K; k0 += BK) {
    // stage A: BK x BM values, 4 per thread
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      int e = tid + u * 256;
      int kk, mm;
      if (trans_a) {  // A is [K, M]: m fastest
        mm = e & 63;
        kk = e >> 6;
      } else {  // A is [M, K]: k fastest
        kk = e & 15;
        mm = e >> 4;
      }
      int m = m0 + mm, k = k0 + kk;
      float v = 0.f;
      if (m < M && k < K) v = to_f32(trans_a ? A[(size_t)k * lda + m] : A[(size_t)m * lda + k]);
      As[kk][mm] = v;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      int e = tid + u * 256;
      int kk, nn;
      if (trans_b) {  // B is [N, K]: k fastest
        kk = e & 15;
        nn = e >> 4;
      } else {  // B is [K, N]: n fastest
        nn = e & 63;
        kk = e >> 6;
      }
      int n = n0 + nn, k = k0 + kk;
      float v = 0.f;
      if (n < N && k < K) v = to_f32(trans_b ? B[(size_t)n * ldb + k] : B[(size_t)k * ldb + n]);
      Bs[kk][nn] = v;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < BK; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[kk][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Bs[kk][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int m = m0 + ty * 4 + i;
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int n = n0 + tx * 4 + j;
      if (n < N) epilogue_store<T>(ep, m, n, acc[i][j]);
    }
  }
}

bool gemm_generic(int dtype, int trans_a, int trans_b, int M, int N, int K, const void* A, int lda, const void* B,
                  int ldb, const Epilogue& ep, hipStream_t stream) {
  if (M <= 0 || N <= 0 || K <= 0 || !A || !B) {
    set_error("gemm: M=%d N=%d K=%d A=%p B=%p", M, N, K, A, B);
    return false;
  }
  int need_lda = trans_a ? M : K, need_ldb = trans_b ? K : N;
  if (lda < need_lda || ldb < need_ldb || ep.ldc < N) {
    set_error("gemm: leading dimensions lda=%d ldb=%d ldc=%d too small for M=%d N=%d K=%d", lda, ldb, ep.ldc, M, N,
              K);
    return false;
  }
  if (!ep.out && !ep.acc_f32) {
    set_error("gemm: no output");
    return false;
  }
  if (ep.gelu_u && !ep.out) {
    set_error("gemm: gelu_u needs out");
    return false;
  }
  dim3 grid(ceil_div(N, 64), ceil_div(M, 64)), block(256);
  if (dtype == kF32)
    gemm_generic_kernel<float><<<grid, block, 0, stream>>>(trans_a, trans_b, M, N, K, (const float*)A, lda,
                                                           (const float*)B, ldb, ep);
  else
    gemm_generic_kernel<bf16><<<grid, block, 0, stream>>>(trans_a, trans_b, M, N, K, (const bf16*)A, lda,
                                                          (const bf16*)B, ldb, ep);
  return launch_ok("gemm_generic_kernel");
}

// Products that stay with the vector kernel: a K that fills no more than a chunk or two (128 bytes of a row each, loaded and
// multiplied whole) under many tiles.  bf16, vector / 64 x 64 matrix-core tiles, us: 1032 x 4104, K 8 / 24 7.9 / 9.6, 10.0 / 9.6; its
// weight gradients have better kernels.  fp32: the line was drawn against 64 x 64 tiles whose waves loaded for themselves (weight
// gradients 4096 x 4096, K 16 / 32 40.8 / 51.0, 48.3 / 51.0) and has not been moved since; the tiles of today are faster on both
// sides of it: 1024 x 512, K 16 / 20 7.5 / 3.4, 9.5 / 3.5; 4096 x 4096, K 16 / 32 / 48 / 52 42 / 35, 49 / 34, 58 / 42, 63 / 42;
// 4096 x 2048, K 32 / 40 31 / 20, 35 / 23.
static bool stays_with_vector_kernel(int dtype, int trans_a, int M, int N, int K) {
  const int64_t tiles = (int64_t)ceil_div(M, 64) * ceil_div(N, 64);
  if (dtype == kBF16) return !trans_a && K <= 16 && tiles >= 1024;
  return K <= 48 && tiles >= (K <= 16 ? 128 : K <= 32 ? 4096 : 2048);
}

bool gemm(int dtype, int trans_a, int trans_b, int M, int N, int K, const void* A, int lda, const void* B, int ldb,
          const Epilogue& ep, bool force_generic, hipStream_t stream) {
  if (force_generic) return gemm_generic(dtype, trans_a, trans_b, M, N, K, A, lda, B, ldb, ep, stream);
  const bool small = gemm_small_supported(dtype, trans_a, trans_b, M, N, K, A, lda, B, ldb) &&
                     !stays_with_vector_kernel(dtype, trans_a, M, N, K);
  if (dtype == kBF16) {
    // bf16 by size.  Whole tiles: the large tiles, or the small ones where those leave most of the chip idle, for the
    // forward and the input gradients (512 x 512, K 512: 11.8 -> 5 us); a weight gradient on its own stays with the large
    // ones, bit for bit what po_op_gemm_grouped gives (a stage's group of few tiles takes the small ones).
    const bool few = small && (trans_a || gemm_mfma_edge_supported(trans_a, trans_b, M, N, K, A, lda, B, ldb, ep)) &&
                     gemm_small_is_faster(M, N, K);
    if (gemm_mfma_supported(trans_a, trans_b, M, N, K, lda, ldb, ep.ldc) && (trans_a || !few))
      return gemm_mfma_bf16(trans_a, trans_b, M, N, K, A, lda, B, ldb, ep, stream);
    if (!few && gemm_mfma_edge_supported(trans_a, trans_b, M, N, K, A, lda, B, ldb, ep))
      return gemm_mfma_edge(trans_a, trans_b, M, N, K, A, lda, B, ldb, ep, stream);
  }
  if (small) return gemm_small(dtype, trans_a, trans_b, M, N, K, A, lda, B, ldb, ep, stream);
  return gemm_generic(dtype, trans_a, trans_b, M, N, K, A, lda, B, ldb, ep, stream);
}

bool gemm_grouped_supported(int dtype, int n, const GemmProblem* p) {
  return gemm_small_grouped_supported(dtype, n, p) ||
         (dtype == kBF16 && (gemm_mfma_grouped_supported(n, p) || gemm_mfma_grouped_edge_supported(n, p)));
}

static bool group_is_small(int dtype, int n, const GemmProblem* p) {
  return gemm_small_grouped_supported(dtype, n, p) &&
         (dtype == kF32 || gemm_small_group_is_faster(n, p) ||
          !(gemm_mfma_grouped_supported(n, p) || gemm_mfma_grouped_edge_supported(n, p)));
}

// The sums' blocks come first and run beside the tiles; what is saved is the launch (or two) and what those took alone.  A block
// sums all rows of its columns, a chain that outlasts the tiles where a bf16 product's K is long.  Two layers of width h and s rows,
// 2 or 4 microbatches, launches of their own / in passing, us: bf16 h 512, s 256 840 / 782, s 512 905 / 843, s 1000
// 1402 / 1329, s 2048 1624 / 1561, s 4096 1467 / 1456, s 8192 1537 / 1553; h 256, s 1024 970 / 922, s 2048 1267 / 1221, s 4096
// 954 / 950, s 8192 1644 / 1673; fp32 h 256, s 128 1086 / 1043, h 1024, s 1024 3228 / 3168, s 2048 6628 / 6544.  The lines lie lower than
// these figures say: they were drawn when a block was slower (bf16 h 512, s 2048 1714 / 1709, s 4096 1556 / 1620) and its fp32 sums had
// a larger error than partial sums from 1100 rows on, and have not been moved since (fp32 bias sums against 64 bits, partial / in
// passing now: 1024 rows 9.4e-8 / 9.0e-8, 1400 10.0e-8 / 9.2e-8, 4096 11.5e-8 / 10.6e-8).
bool gemm_grouped_takes_sums(int dtype, int n, const GemmProblem* p, const ReduceJob* jobs, int n_jobs, int rows) {
  int64_t blocks = 0;  // at most, of at most 640 threads: a grid of one dimension
  for (int j = 0; j < n_jobs; ++j) blocks += ceil_div(jobs[j].n, 32);
  for (int i = 0; i < n; ++i) blocks += (int64_t)ceil_div(p[i].M, 32) * ceil_div(p[i].N, 32);
  return rows <= (dtype == kF32 ? 1024 : 1536) && blocks * 640 < (int64_t)1 << 31 && group_is_small(dtype, n, p) &&
         column_sums_vectors(dtype, jobs, n_jobs);
}

bool gemm_grouped_accumulate_with_sums(int dtype, int n, const GemmProblem* p, const ReduceJob* jobs, int n_jobs, int rows,
                                       hipStream_t stream) {
  return gemm_small_grouped_accumulate(dtype, n, p, stream, jobs, n_jobs, rows);
}

bool gemm_grouped_accumulate(int dtype, int n, const GemmProblem* p, hipStream_t stream) {
  if (dtype == kBF16 && !group_is_small(dtype, n, p)) {
    if (gemm_mfma_grouped_supported(n, p)) return gemm_mfma_grouped_accumulate(n, p, stream);
    if (gemm_mfma_grouped_edge_supported(n, p)) return gemm_mfma_grouped_edge_accumulate(n, p, stream);
  }
  return gemm_small_grouped_accumulate(dtype, n, p, stream);
}

}  // namespace po
