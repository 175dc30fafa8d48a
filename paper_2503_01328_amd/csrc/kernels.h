// Host-side launchers of the HIP kernels.  Every launcher validates its shapes
// on the host, enqueues on `stream`, and returns false with po::set_error text
// when the arguments do not fit what the kernel assumes.
#pragma once

#include <atomic>

#include "po_common.h"

namespace po {

void set_error(const char* fmt, ...);
const char* get_error();

// ---- elementwise / normalisation (elementwise.hip) -------------------------
// copy (may be null): where x goes too.
bool layernorm_forward(int dtype, const void* x, const void* gain, const void* shift, void* y, int rows, int h,
                       float eps, hipStream_t stream, void* copy = nullptr);
size_t layernorm_backward_workspace(int rows, int h);
// parts: kLnInputGrad writes dx (= dres + LayerNorm input gradient) and the row statistics into the workspace;
// kLnParamGrad adds the gain / shift gradients, reading the statistics an earlier or the same call left there.
// n_out (with shift, kLnInputGrad only): also writes LayerNorm(x), bit for bit what layernorm_forward writes, for a
// caller that needs the recomputed forward output next and would otherwise read x once more for it.
enum { kLnInputGrad = 1, kLnParamGrad = 2 };
bool layernorm_backward(int dtype, const void* dn, const void* x, const void* gain, const void* dres, void* dx,
                        float* dgain, float* dshift, float* workspace, int rows, int h, float eps, int parts,
                        hipStream_t stream, const void* shift = nullptr, void* n_out = nullptr);
size_t colsum_workspace(int rows, int n);
bool colsum_accumulate(int dtype, const void* x, float* acc, float* workspace, int rows, int n, hipStream_t stream);
// The same with the partials in a device array built into the library (no workspace, nothing allocated);
// n <= 32768.  Calls that overlap on one GPU share that array and race.
bool colsum_accumulate_static(int dtype, const void* x, float* acc, int rows, int n, hipStream_t stream);
// Several column reductions over the same number of rows in one launch or two (all partial sums, then all final
// sums) instead of as many per tensor: the bias gradients and LayerNorm gain / shift gradients of one layer.
// colsum_accumulate and layernorm_backward(kLnParamGrad) are such reductions of one tensor.
struct ReduceJob {
  const void* a;       // [rows, n] of dtype: the tensor summed over rows, or dn of a LayerNorm
  const void* x;       // LayerNorm input [rows, n]; null: plain column sum
  const float* stats;  // LayerNorm row statistics [rows][2] (mean, 1/std) left by kLnInputGrad; null for a sum
  float* out0;         // [n] fp32, += column sum, or += gain gradient
  float* out1;         // [n] fp32, += shift gradient (LayerNorm only)
  float* partials;     // fp32 workspace: column_reductions_workspace(rows, n) floats, x2 for a LayerNorm job
  int n;               // columns, even
};
constexpr int kMaxReduceJobs = 8;
size_t column_reductions_workspace(int rows, int n);  // bytes per output plane
bool column_reductions(int dtype, const ReduceJob* jobs, int n_jobs, int rows, hipStream_t stream);
bool embedding_forward(int dtype, const int32_t* tok, const void* wte, const void* wpe, void* x, int s, int h,
                       int vocab, hipStream_t stream);
bool embedding_backward(int dtype, const int32_t* tok, const void* dx, float* dwte, float* dwpe, int s, int h,
                        int vocab, hipStream_t stream);
bool fill_u32(void* p, uint32_t pattern, size_t bytes, hipStream_t stream);

constexpr int kMaxPackSegments = 48;
bool pack_segments(const void* const* seg_ptrs, const uint64_t* seg_bytes, int n_seg, void* packed,
                   hipStream_t stream);
bool unpack_segments(void* const* seg_ptrs, const uint64_t* seg_bytes, int n_seg, const void* packed,
                     hipStream_t stream);

// ---- GEMM (gemm_generic.hip, gemm_mfma.hip) ---------------------------------
// C[M,N] = op(A) op(B): trans_a == 0: A [M,K] (lda >= K); 1: A [K,M] (lda >= M).
// trans_b == 0: B [K,N] (ldb >= N); 1: B [N,K] (ldb >= K).
bool gemm_generic(int dtype, int trans_a, int trans_b, int M, int N, int K, const void* A, int lda, const void* B,
                  int ldb, const Epilogue& ep, hipStream_t stream);
// bf16 MFMA path; returns false (with error text) if the shape is not supported.
bool gemm_mfma_supported(int trans_a, int trans_b, int M, int N, int K, int lda, int ldb, int ldc);
// Output tile (rows, columns) the bf16 MFMA path uses for an M x N result; 0, 0 if it has none for the shape.
void gemm_mfma_tile(int M, int N, int* bm, int* bn);
bool gemm_mfma_bf16(int trans_a, int trans_b, int M, int N, int K, const void* A, int lda, const void* B, int ldb,
                    const Epilogue& ep, hipStream_t stream);
// Several weight-gradient GEMMs in one launch, C_i [M_i, N_i] (fp32) += A_i^T B_i with A_i [K_i, M_i] and
// B_i [K_i, N_i] bf16: the form of the four parameter-gradient products of a layer.  Supported when every M_i and
// N_i is a multiple of 256 and every K_i of 64 (at most 4 problems); results equal the single launches bit for bit.
struct GemmProblem {
  int M, N, K;
  const void* A;
  int lda;
  const void* B;
  int ldb;
  float* acc_f32;
  int ldc;
};
bool gemm_mfma_grouped_supported(int n, const GemmProblem* p);
bool gemm_mfma_grouped_accumulate(int n, const GemmProblem* p, hipStream_t stream);
// The same kernels for results that are no whole tiles (gemm_mfma.hip, `edge`): the three forms a layer uses, M any and N a
// multiple of 8, K of 64 (weight gradients: M of 8, K any), 16-byte alignment of everything.
bool gemm_mfma_edge_supported(int trans_a, int trans_b, int M, int N, int K, const void* A, int lda, const void* B,
                              int ldb, const Epilogue& ep);
bool gemm_mfma_edge(int trans_a, int trans_b, int M, int N, int K, const void* A, int lda, const void* B, int ldb,
                    const Epilogue& ep, hipStream_t stream);
bool gemm_mfma_grouped_edge_supported(int n, const GemmProblem* p);
bool gemm_mfma_grouped_edge_accumulate(int n, const GemmProblem* p, hipStream_t stream);
// Whether the 64 x 64 and 32 x 32 tiles of gemm_small.hip beat the large ones for a bf16 product (a group of them).
bool gemm_small_is_faster(int M, int N, int K);
bool gemm_small_group_is_faster(int n, const GemmProblem* p);
// Matrix-core kernel for fp32 and for bf16 shapes of any size (gemm_small.hip): rows of both operands whole 16-byte
// vectors, operands 16-byte aligned.
bool gemm_small_supported(int dtype, int trans_a, int trans_b, int M, int N, int K, const void* A, int lda,
                          const void* B, int ldb);
bool gemm_small(int dtype, int trans_a, int trans_b, int M, int N, int K, const void* A, int lda, const void* B,
                int ldb, const Epilogue& ep, hipStream_t stream);
// The counterpart of gemm_mfma_grouped_accumulate for its shapes and types.
bool gemm_small_grouped_supported(int dtype, int n, const GemmProblem* p);
// jobs: column sums over `rows` rows that the same launch does (column_sums_vectors).
bool gemm_small_grouped_accumulate(int dtype, int n, const GemmProblem* p, hipStream_t stream,
                                   const ReduceJob* jobs = nullptr, int n_jobs = 0, int rows = 0);
// Several weight-gradient products in one launch of whichever of those kernels takes them and is the fastest.
bool gemm_grouped_supported(int dtype, int n, const GemmProblem* p);
bool gemm_grouped_accumulate(int dtype, int n, const GemmProblem* p, hipStream_t stream);
// Whether that launch does a layer's column sums in passing (gemm_grouped_accumulate_with_sums), and cheaper than
// column_reductions would.  The sums come out the same up to the order of additions.
bool gemm_grouped_takes_sums(int dtype, int n, const GemmProblem* p, const ReduceJob* jobs, int n_jobs, int rows);
bool gemm_grouped_accumulate_with_sums(int dtype, int n, const GemmProblem* p, const ReduceJob* jobs, int n_jobs, int rows,
                                       hipStream_t stream);
// Picks the kernel by type and shape; force_generic: the vector kernel.
bool gemm(int dtype, int trans_a, int trans_b, int M, int N, int K, const void* A, int lda, const void* B, int ldb,
          const Epilogue& ep, bool force_generic, hipStream_t stream);

// ---- dropout with regenerated masks (elementwise.hip) --------------------------
// threshold = round(p 2^32) (an element is kept iff its random word is >= it), scale = 1 / (1 - p), key = seed.
DropoutSite make_dropout_site(float p, uint64_t seed, int layer, int site, int unit);
// out = (residual ? residual : 0) + dropout(x); x, residual, out are [rows, cols] of dtype.
bool dropout_apply(int dtype, const void* x, const void* residual, void* out, int rows, int cols,
                   const DropoutSite& d, hipStream_t stream);

// ---- attention (attention_generic.hip, attention_mfma.hip) -------------------
// qkv is [s, h + 2 hkv]: query block [h], key block [hkv], value block [hkv], hkv = n_kv_heads * (h / n_heads);
// query head t reads key/value head t / (n_heads / n_kv_heads).  n_kv_heads = n_heads is plain multi-head.
bool attention_forward_generic(int dtype, const void* qkv, void* o, float* lse, int s, int h, int n_heads,
                               int n_kv_heads, hipStream_t stream);
bool attention_backward_generic(int dtype, const void* qkv, const void* o, const float* lse, const void* d_o,
                                void* dqkv, float* delta, int s, int h, int n_heads, int n_kv_heads,
                                hipStream_t stream);
// fp32 on the matrix cores (attention_f32.hip): head sizes 32, 64, 96, 128, 16-byte aligned tensors.  The backward takes
// delta as given; attention_delta_f32 forms it, by whole vectors.
bool attention_f32_supported(const void* qkv, const void* o, int s, int h, int n_heads, int n_kv_heads);
bool attention_forward_f32(const float* qkv, float* o, float* lse, int s, int h, int n_heads, int n_kv_heads,
                           hipStream_t stream);
bool attention_backward_f32(const float* qkv, const float* lse, const float* delta, const float* d_o, float* dqkv, int s,
                            int h, int n_heads, int n_kv_heads, hipStream_t stream);
bool attention_delta_f32(const float* o, const float* d_o, float* delta, int s, int h, int n_heads, hipStream_t stream);
bool attention_mfma_supported(int s, int h, int n_heads, int n_kv_heads);
bool attention_forward_mfma(const void* qkv, void* o, float* lse, int s, int h, int n_heads, int n_kv_heads,
                            hipStream_t stream);
// partials: optional workspace of 4 s h bytes; with it, grouped-query shapes with few key/value heads run dK/dV per query head
// (s a multiple of 128: bf16 partials) or per two query heads or the group's next divisor (else: fp32 partials, if it is
// 16-byte aligned and the group has such a divisor) and add the groups up afterwards.
bool attention_backward_mfma(const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv,
                             float* delta, void* partials, int s, int h, int n_heads, int n_kv_heads,
                             hipStream_t stream);
// bf16 in blocks of 32 rows (attention_few.hip) for launches that blocks of 128 rows would leave most of the chip idle: shapes and
// pointers that attention_*_mfma have checked, where *_is_faster says so.  The backward takes delta as given.
bool attention_few_forward_is_faster(int s, int h, int n_heads, int n_kv_heads);
bool attention_few_forward(const bf16* qkv, bf16* o, float* lse, int s, int h, int n_heads, int n_kv_heads,
                           hipStream_t stream);
// A dK/dV block walks hpb query heads; partials: null (hpb is the whole group), or where their fp32 results go.
bool attention_few_backward_is_faster(int s, int h, int n_heads, int n_kv_heads, int hpb);
bool attention_few_backward(const bf16* qkv, const float* lse, const float* delta, const bf16* d_o, bf16* dqkv,
                            float* partials, int hpb, int s, int h, int n_heads, int n_kv_heads, hipStream_t stream);
bool attention_forward(int dtype, const void* qkv, void* o, float* lse, int s, int h, int n_heads, int n_kv_heads,
                       bool force_generic, hipStream_t stream);
bool attention_backward(int dtype, const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv,
                        float* delta, void* partials, int s, int h, int n_heads, int n_kv_heads, bool force_generic,
                        hipStream_t stream);

#define PO_HIP_OK(expr)                                                                  \
  do {                                                                                   \
    hipError_t e__ = (expr);                                                             \
    if (e__ != hipSuccess) {                                                             \
      po::set_error("%s failed: %s (%s:%d)", #expr, hipGetErrorString(e__), __FILE__, __LINE__); \
      return false;                                                                      \
    }                                                                                    \
  } while (0)

// Blocks in the second dimension of a grid.  The attention kernels that tile the rows there leave longer sequences to the
// vector kernels, which have them in the first.
constexpr int kMaxGridY = 65535;

// The dynamic LDS a kernel may ask for: set once per kernel (a static object beside its launch) and device.  A call that
// fails leaves its error text and the next one tries again.
class LdsLimit {
  std::atomic<uint64_t> devices_{0};  // one bit per device it has been set on

 public:
  template <typename Kernel>
  bool allow(Kernel kern, int bytes) {
    int device = 0;
    PO_HIP_OK(hipGetDevice(&device));
    const uint64_t bit = device < 64 ? (uint64_t)1 << device : 0;
    if (devices_.load(std::memory_order_relaxed) & bit) return true;
    PO_HIP_OK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
    devices_.fetch_or(bit, std::memory_order_relaxed);
    return true;
  }
};

// hipGetLastError is sticky per thread: an error left behind by an earlier, unrelated HIP call
// (of this library or of the host program) must not be blamed on the next launch.
inline void begin_launch() { (void)hipGetLastError(); }

inline bool launch_ok(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error("launch of %s failed: %s", what, hipGetErrorString(e));
    return false;
  }
  return true;
}

}  // namespace po
