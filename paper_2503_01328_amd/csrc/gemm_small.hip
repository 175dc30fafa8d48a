// GEMM on the matrix cores for any M, N, K and for fp32 as well as bf16: the kernel of short or narrow operands whose larger
// tiles (gemm_mfma.hip; gemm_f32.hip for fp32) would leave most of the chip idle, and of every bf16 product that is no multiple of
// a tile.
//
// A block owns a (32 TM) x (32 TN) tile of C and has KG waves.  Every wave owns the WHOLE tile for every KG-th chunk
// of K (128 bytes of a row: 64 bf16 or 32 fp32), so the waves never wait for each other in the main loop: each has
// its own ring of two LDS stages that it fills (HBM -> LDS directly) and reads alone, with waits on its own load counter
// and no barrier at all.  A small product is a chain of memory round trips; KG of them run side by side here.  The
// KG partial tiles are added in wave order through LDS at the end (always the same order: deterministic).
//
// fp32 runs on v_mfma_f32_32x32x2_f32 (full fp32 products and sums, 256 flop/clk/CU), bf16 on
// v_mfma_f32_32x32x16_bf16.  The k-index a lane feeds to an fp32 MFMA is permuted the same way for both operands
// (half-wave h takes k = 8 kk + 4 h + j in step j) so that four steps' operands are one 16-byte read.
//
// Edges: operands are loaded through buffer descriptors that end with the operand, so rows past M or N and, for
// operands stored k-major, k past K read as zero; for k-contiguous operands the last chunk's lanes past K point past
// the end.  The epilogue stores only what is inside.
#include <string.h>

#include "gemm_tile.h"

namespace po {

template <typename T, int TM, int TN, int KG, bool TA, bool TB>
__device__ __forceinline__ void small_tile(const SmallProblem& p, int tile, char* smem) {
  constexpr int BM = 32 * TM, BN = 32 * TN, KU = MfmaOf<T>::KU;
  static_assert(BM <= kMaxSmallRows && BN <= kMaxSmallRows, "gemm_small_supported bounds a lane's offset");
  using OpA = Operand<T, BM, TA>;
  using OpB = Operand<T, BN, TB>;
  constexpr int STAGE = OpA::BYTES + OpB::BYTES, LOADS = OpA::LOADS + OpB::LOADS;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int M = p.M, N = p.N, K = p.K;
  int m0, n0;
  place_of_tile(tile, (M + BM - 1) / BM, p.tiles_n, m0, n0);
  m0 *= BM;
  n0 *= BN;

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  const int chunks = (K + KU - 1) / KU;
  const int mine = chunks > wave ? (chunks - wave + KG - 1) / KG : 0;  // chunks wave, wave + KG, ...
  OpA a;
  OpB b;
  a.init(static_cast<const T*>(p.A), p.lda, m0, M, K, wave, KG, lane);
  b.init(static_cast<const T*>(p.B), p.ldb, n0, N, K, wave, KG, lane);
  char* ring = smem + wave * (2 * STAGE);
  const unsigned ring_lds = __builtin_amdgcn_readfirstlane((int)lds_byte(ring));
  auto issue = [&](int t) {
    int k_left = K - (wave + t * KG) * KU;
    unsigned dst = ring_lds + (t & 1) * STAGE;
    a.issue(dst, k_left, lane);
    b.issue(dst + OpA::BYTES, k_left, lane);
  };
  if (mine > 0) issue(0);
  if (mine > 1) issue(1);
  for (int t = 0; t < mine; ++t) {
    if (t + 1 < mine) wait_loads<LOADS>();
    else wait_loads<0>();
    const char* sa = ring + (t & 1) * STAGE;
    const char* sb = sa + OpA::BYTES;
    using Frag = decltype(fragment<BM, TA>((const T*)nullptr, sa, 0, 0, lane));
    Frag fa[4][TM], fb[4][TN];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[kk][i] = fragment<BM, TA>((const T*)nullptr, sa, 32 * i, kk, lane);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[kk][j] = fragment<BN, TB>((const T*)nullptr, sb, 32 * j, kk, lane);
    }
    // the stage is free once its fragments are in registers: the chunk after next is requested before the MFMAs
    wait_lds_reads();
    __builtin_amdgcn_sched_barrier(0);
    if (t + 2 < mine) issue(t + 2);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = multiply(fb[kk][j], fa[kk][i], acc[i][j]);
  }

  // Partial tiles side by side in LDS (each wave in its own ring), then every thread adds its pieces in wave order.
  constexpr int LD = BN + 4;
  static_assert(BM * LD * 4 <= 2 * STAGE, "a partial tile fits the wave's ring");
  float* part = reinterpret_cast<float*>(ring);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        f32x4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
        *reinterpret_cast<f32x4*>(part + (32 * i + (lane & 31)) * LD + 32 * j + 8 * q + 4 * (lane >> 5)) = v;
      }
  __syncthreads();
  constexpr int V = Vec16<T>::N, PER_ROW = BN / V;
  for (int piece = threadIdx.x; piece < BM * PER_ROW; piece += 64 * KG) {
    int r = piece / PER_ROW, c = piece % PER_ROW * V;
    if (m0 + r >= M || n0 + c >= N) continue;
    float v[V];
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] = 0.f;
#pragma unroll
    for (int g = 0; g < KG; ++g)
#pragma unroll
      for (int i = 0; i < V; i += 4) {
        f32x4 w = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(smem + g * (2 * STAGE)) + r * LD + c + i);
#pragma unroll
        for (int k = 0; k < 4; ++k) v[i + k] += w[k];
      }
    if (p.vec && n0 + c + V <= N) {
      epilogue_vector<T>(p.ep, m0 + r, n0 + c, v);
    } else {
#pragma unroll
      for (int i = 0; i < V; ++i)
        if (n0 + c + i < N) epilogue_store<T>(p.ep, m0 + r, n0 + c + i, v[i]);
    }
  }
}

template <typename T, int TM, int TN, int KG, bool TA, bool TB>
__global__ __launch_bounds__(64 * KG) void gemm_small_kernel(SmallProblem p) {
  extern __shared__ __align__(16) char smem[];
  small_tile<T, TM, TN, KG, TA, TB>(p, tile_of_block(), smem);
}

// fp32 results of so few tiles that a CU's four SIMDs would be a chain of MFMAs each: tiles of 16 x 16 with eight waves, four
// times the blocks, a quarter of the MFMAs per wave.  Four stages a wave: up to K 1024 all of its chunks are on their way at
// once.  Otherwise as above; every sum in eight chains.
template <bool TA, bool TB>
__global__ __launch_bounds__(512) void gemm_tiny_f32_kernel(SmallProblem p) {
  constexpr int KG = 8, NS = 4, KU = MfmaOf<float>::KU, LD = 16 + 4;
  using OpA = Operand<float, 16, TA>;
  using OpB = Operand<float, 16, TB>;
  constexpr int STAGE = OpA::BYTES + OpB::BYTES, LOADS = OpA::LOADS + OpB::LOADS;
  static_assert(16 * LD * 4 <= NS * STAGE, "a partial tile fits the wave's ring");
  extern __shared__ __align__(16) char smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int m0, n0;
  place_of_tile(tile_of_block(), (p.M + 15) / 16, p.tiles_n, m0, n0);
  m0 *= 16;
  n0 *= 16;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  const int chunks = (p.K + KU - 1) / KU, mine = chunks > wave ? (chunks - wave + KG - 1) / KG : 0;
  OpA a;
  OpB b;
  a.init(static_cast<const float*>(p.A), p.lda, m0, p.M, p.K, wave, KG, lane);
  b.init(static_cast<const float*>(p.B), p.ldb, n0, p.N, p.K, wave, KG, lane);
  char* ring = smem + wave * (NS * STAGE);
  const unsigned ring_lds = __builtin_amdgcn_readfirstlane((int)lds_byte(ring));
  auto issue = [&](int t) {
    const int k_left = p.K - (wave + t * KG) * KU;
    const unsigned dst = ring_lds + t % NS * STAGE;
    a.issue(dst, k_left, lane);
    b.issue(dst + OpA::BYTES, k_left, lane);
  };
#pragma unroll
  for (int t = 0; t < NS; ++t)
    if (t < mine) issue(t);
  for (int t = 0; t < mine; ++t) {
    const int behind = mine - 1 - t;  // chunks that may still be on their way, up to NS - 1
    if (behind >= 3) wait_loads<3 * LOADS>();
    else if (behind == 2) wait_loads<2 * LOADS>();
    else if (behind == 1) wait_loads<LOADS>();
    else wait_loads<0>();
    const char* sa = ring + t % NS * STAGE;
    f32x4 fa[2], fb[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      fa[kk] = fragment16<TA>(sa, kk, lane);
      fb[kk] = fragment16<TB>(sa + OpA::BYTES, kk, lane);
    }
    wait_lds_reads();
    __builtin_amdgcn_sched_barrier(0);
    if (t + NS < mine) issue(t + NS);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[kk][j], fa[kk][j], acc, 0, 0, 0);
  }
  // lane: row lane % 16, columns 4 (lane / 16) .. + 3
  *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(ring) + (lane & 15) * LD + 4 * (lane >> 4)) = acc;
  __syncthreads();
  const int r = threadIdx.x >> 2, c = (threadIdx.x & 3) * 4;
  if (r >= 16 || m0 + r >= p.M || n0 + c >= p.N) return;
  float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int g = 0; g < KG; ++g) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(smem + g * (NS * STAGE)) + r * LD + c);
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] += x[k];
  }
  if (p.vec && n0 + c + 4 <= p.N) {
    epilogue_vector<float>(p.ep, m0 + r, n0 + c, v);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (n0 + c + i < p.N) epilogue_store<float>(p.ep, m0 + r, n0 + c + i, v[i]);
  }
}

// Columns of a column-sum block: half of the 64 where a block has few waves, each of whose rounds over the rows is a chain of
// memory round trips.
template <int KG>
constexpr int kSumColumns = KG <= 2 ? 32 : 64;

// The four weight-gradient products of a layer in one launch: the tiles of all of them one product after the other.
template <typename T, int TM, int TN, int KG>
__device__ __forceinline__ void small_group_tile(const SmallGroup& g, int lin, char* smem) {
  SmallProblem p = g.p[0];  // constant indices only: a run-time index would send the arguments through memory
#pragma unroll
  for (int i = 1; i < kMaxSmallGroup; ++i)
    if (i < g.n && lin >= g.p[i].first_tile) p = g.p[i];
  small_tile<T, TM, TN, KG, true, true>(p, lin - p.first_tile, smem);
}
template <typename T, int TM, int TN, int KG>
__global__ __launch_bounds__(64 * KG) void gemm_small_grouped_kernel(SmallGroup g) {
  extern __shared__ __align__(16) char smem[];
  small_group_tile<T, TM, TN, KG>(g, tile_of_block(), smem);
}
// And its column sums, in blocks of their own before the others, which hide them.
template <typename T, int TM, int TN, int KG>
__global__ __launch_bounds__(64 * KG) void gemm_small_with_sums_kernel(SmallGroup g, GroupSums sums) {
  extern __shared__ __align__(16) char smem[];
  if ((int)blockIdx.x < sums.blocks)
    column_sums_block<T, 64 * KG, kSumColumns<KG>, 4>(sums.batch, blockIdx.x, sums.rows, reinterpret_cast<float*>(smem));
  else
    small_group_tile<T, TM, TN, KG>(g, tile_of_block(sums.blocks), smem);
}

// ---- host side -------------------------------------------------------------------------------------------------
// Waves of a block and its tile.  Times in us of one launch with warm operands, forms 32x32 with 8 and 4 waves, 64x64
// with 4, 2 and 1 waves:
//   bf16  512 x  512, K  512:  3.8  3.6   5.0   5.8   8.6        bf16  512 x 1536, K  512:  8.9  6.3  5.1  5.9  8.7
//   bf16  512 x  512, K 2048:  7.5  6.1   9.0  12.8  21.8        bf16 1024 x 1024, K 1024: 13.4  9.6  6.7  8.3 13.3
//   bf16  100 x 2048, K 8192: 19.0 19.4  25.3  39.9  73.7        bf16  100 x 8192, K 2048: 22.2 17.7 10.7 13.3 22.0
//   bf16 2048 x 2048, K  100: 30.0 16.3  14.6  11.2   9.8        bf16 1733 x 6144, K 2048:  207  140   86   76   72
//   fp32  128 x  256, K 1024:  8.0  8.3  21.0  37.8  72.2 (16 x 16: 5.1)
// A 32 x 32 tile halves what an operand byte is used for but makes four times as many blocks: it wins while 64 x 64
// tiles leave half of the CUs without one.  From there on more waves per tile shorten its chain of chunks, as long as
// every wave has a few chunks and the chip is not full anyway: bf16 has as many as keep four waves on every CU.  fp32 has
// 32 x 32 tiles alone, with eight waves where those have two chunks each.
struct SmallForm {
  int edge, waves;
};
static SmallForm small_form(int dtype, int64_t tiles64, int K) {
  if (dtype == kF32) return {32, K > 15 * 32 ? 8 : 4};
  if (tiles64 < 128) return {32, 4};
  int waves = tiles64 < 512 ? 4 : tiles64 < 1024 ? 2 : 1;
  while (waves > 1 && ceil_div(K, 64) < 2 * waves) waves /= 2;
  return {64, waves};
}
// fp32 results for which 32 x 32 tiles beat the larger ones of gemm_f32.hip: few enough for one round of the CUs (a short K
// is over before a larger tile's first chunks have arrived).  32 x 32 / best larger, us, 32 x 32 tiles in brackets:
//   300 x 512, K 512 5.4 / 8.2 (160); 356 x 652, K 1844 15.1 / 20.3 (252); 1272 x 216, K 228 5.4 / 6.3 (280);
//   636 x 496, K 316 6.8 / 6.8 (320); 516 x 712, K 772 13.4 / 11.3 (391); 680 x 572, K 68 3.9 / 5.2 (396)
static bool f32_few_tiles(int64_t tiles32, int K) { return tiles32 <= 288 || (tiles32 < 448 && K < 128); }

// fp32 results for which 16 x 16 tiles beat 32 x 32 ones: as many as one round of the CUs.  A 32 x 32 x 32 chunk is 1024 cycles of
// MFMAs on its SIMD, and few tiles leave most of the chip idle.  32 x 32 / 16 x 16, us, 16 x 16 tiles in brackets:
//   128 x 256, K 256 4.0 / 3.4 (128); 64 x 128, K 512 5.2 / 3.9 (32); 128 x 256, K 1024 7.9 / 5.1 (128); 256 x 256, K 1024 7.9 / 5.4 (256);
//   128 x 512, K 2048 12.5 / 7.7 (256); 128 x 256, K 4096 21.4 / 10.9 (128); 200 x 320, K 1280 9.0 / 9.6 (260); 128 x 768, K 256
//   4.0 / 5.3 (384).  Against 64 bits the same, at K 256 1.18e-7 instead of 1.50e-7 (eight chains instead of four).
static bool f32_tiny(int M, int N) { return (int64_t)ceil_div(M, 16) * ceil_div(N, 16) <= 256; }

static bool vector_epilogue(int dtype, const Epilogue& ep) {
  const int v = dtype == kF32 ? 4 : 8;
  return ep.ldc % v == 0 && ((uintptr_t)ep.bias | (uintptr_t)ep.residual | (uintptr_t)ep.out | (uintptr_t)ep.gelu_out |
                             (uintptr_t)ep.gelu_u | (uintptr_t)ep.acc_f32) % 16 == 0;
}

bool gemm_small_supported(int dtype, int trans_a, int trans_b, int M, int N, int K, const void* A, int lda,
                          const void* B, int ldb) {
  const int v = dtype == kF32 ? 4 : 8;  // elements of a 16-byte load
  // rows of both operands are whole 16-byte pieces; a lane's offset (less than kMaxSmallRows rows of up to 4 bytes an element)
  // fits 32 bits and the largest buffer
  const int64_t limit = (int64_t)1 << 32;
  return M > 0 && N > 0 && K > 0 && lda % v == 0 && ldb % v == 0 && (trans_a ? M : K) % v == 0 &&
         (trans_b ? K : N) % v == 0 && ((uintptr_t)A | (uintptr_t)B) % 16 == 0 && (int64_t)lda * kMaxSmallRows * 4 < limit &&
         (int64_t)ldb * kMaxSmallRows * 4 < limit;
}

template <typename T, int TM, int TN, int KG, bool TA, bool TB>
static bool launch_small(SmallProblem& p, hipStream_t stream) {
  constexpr int smem = KG * 2 * 32 * (TM + TN) * 128;
  auto kern = gemm_small_kernel<T, TM, TN, KG, TA, TB>;
  static LdsLimit lds;  // per instantiation
  if (!lds.allow(kern, smem)) return false;
  p.tiles_n = ceil_div(p.N, 32 * TN);
  kern<<<ceil_div(p.M, 32 * TM) * p.tiles_n, 64 * KG, smem, stream>>>(p);
  return launch_ok("gemm_small_kernel");
}

template <typename T, int TM, int TN, int KG>
static bool launch_trans(int ta, int tb, SmallProblem& p, hipStream_t stream) {
  // kernel flag TB means "B is n-contiguous", i.e. trans_b == 0
  if (!ta && !tb) return launch_small<T, TM, TN, KG, false, true>(p, stream);
  if (!ta && tb) return launch_small<T, TM, TN, KG, false, false>(p, stream);
  if (ta && !tb) return launch_small<T, TM, TN, KG, true, true>(p, stream);
  return launch_small<T, TM, TN, KG, true, false>(p, stream);
}

template <bool TA, bool TB>
static bool launch_tiny(SmallProblem& p, hipStream_t stream) {
  constexpr int smem = 8 * 4 * 2 * 16 * 128;
  static LdsLimit lds;  // per instantiation
  if (!lds.allow(gemm_tiny_f32_kernel<TA, TB>, smem)) return false;
  p.tiles_n = ceil_div(p.N, 16);
  gemm_tiny_f32_kernel<TA, TB><<<ceil_div(p.M, 16) * p.tiles_n, 512, smem, stream>>>(p);
  return launch_ok("gemm_tiny_f32_kernel");
}
static bool launch_tiny_trans(int ta, int tb, SmallProblem& p, hipStream_t stream) {
  if (!ta && !tb) return launch_tiny<false, true>(p, stream);
  if (!ta && tb) return launch_tiny<false, false>(p, stream);
  if (ta && !tb) return launch_tiny<true, true>(p, stream);
  return launch_tiny<true, false>(p, stream);
}

static bool launch_form(int dtype, SmallForm f, int ta, int tb, SmallProblem& p, hipStream_t stream) {
  if (dtype == kF32)
    return f.waves == 8 ? launch_trans<float, 1, 1, 8>(ta, tb, p, stream) : launch_trans<float, 1, 1, 4>(ta, tb, p, stream);
  if (f.edge == 32) return launch_trans<bf16, 1, 1, 4>(ta, tb, p, stream);
  if (f.waves == 4) return launch_trans<bf16, 2, 2, 4>(ta, tb, p, stream);
  if (f.waves == 2) return launch_trans<bf16, 2, 2, 2>(ta, tb, p, stream);
  return launch_trans<bf16, 2, 2, 1>(ta, tb, p, stream);
}

bool gemm_small(int dtype, int ta, int tb, int M, int N, int K, const void* A, int lda, const void* B, int ldb,
                const Epilogue& ep, hipStream_t stream) {
  int need_lda = ta ? M : K, need_ldb = tb ? K : N;
  if (!gemm_small_supported(dtype, ta, tb, M, N, K, A, lda, B, ldb) || !A || !B || lda < need_lda || ldb < need_ldb ||
      ep.ldc < N || (!ep.out && !ep.acc_f32) || (ep.gelu_u && !ep.out)) {
    set_error("gemm: bad operands M=%d N=%d K=%d A=%p lda=%d B=%p ldb=%d ldc=%d", M, N, K, A, lda, B, ldb, ep.ldc);
    return false;
  }
  SmallProblem p{A, B, ep, M, N, K, lda, ldb, 0, 0, vector_epilogue(dtype, ep)};
  if (dtype == kF32 && f32_tiny(M, N)) return launch_tiny_trans(ta, tb, p, stream);
  if (dtype == kF32 && !f32_few_tiles((int64_t)ceil_div(M, 32) * ceil_div(N, 32), K)) return gemm_f32(ta, tb, p, stream);
  SmallForm f = small_form(dtype, (int64_t)ceil_div(M, 64) * ceil_div(N, 64), K);
  return launch_form(dtype, f, ta, tb, p, stream);
}

template <typename T, int TM, int TN, int KG>
static bool launch_group(SmallGroup& g, GroupSums* sums, hipStream_t stream) {
  constexpr int smem = KG * 2 * 32 * (TM + TN) * 128;
  int total = 0;
  for (int i = 0; i < g.n; ++i) {
    g.p[i].tiles_n = ceil_div(g.p[i].N, 32 * TN);
    g.p[i].first_tile = total;
    total += ceil_div(g.p[i].M, 32 * TM) * g.p[i].tiles_n;
  }
  if (sums) {
    auto kern = gemm_small_with_sums_kernel<T, TM, TN, KG>;
    static LdsLimit lds;
    if (!lds.allow(kern, smem)) return false;
    sums->blocks *= 64 / kSumColumns<KG>;
    kern<<<total + sums->blocks, 64 * KG, smem, stream>>>(g, *sums);
    return launch_ok("gemm_small_with_sums_kernel");
  }
  auto kern = gemm_small_grouped_kernel<T, TM, TN, KG>;
  static LdsLimit lds;
  if (!lds.allow(kern, smem)) return false;
  kern<<<total, 64 * KG, smem, stream>>>(g);
  return launch_ok("gemm_small_grouped_kernel");
}

static bool group_form(int dtype, SmallForm f, SmallGroup& g, GroupSums* sums, hipStream_t stream) {
  if (dtype == kF32)
    return f.waves == 8 ? launch_group<float, 1, 1, 8>(g, sums, stream) : launch_group<float, 1, 1, 4>(g, sums, stream);
  if (f.edge == 32) return launch_group<bf16, 1, 1, 4>(g, sums, stream);
  if (f.waves == 4) return launch_group<bf16, 2, 2, 4>(g, sums, stream);
  if (f.waves == 2) return launch_group<bf16, 2, 2, 2>(g, sums, stream);
  return launch_group<bf16, 2, 2, 1>(g, sums, stream);
}

bool gemm_small_grouped_supported(int dtype, int n, const GemmProblem* prob) {
  if (n < 1 || n > kMaxSmallGroup) return false;
  for (int i = 0; i < n; ++i) {
    const GemmProblem& q = prob[i];
    if (!gemm_small_supported(dtype, 1, 0, q.M, q.N, q.K, q.A, q.lda, q.B, q.ldb) || !q.A || !q.B || !q.acc_f32 ||
        q.lda < q.M || q.ldb < q.N || q.ldc < q.N)
      return false;
  }
  return true;
}

bool gemm_small_grouped_accumulate(int dtype, int n, const GemmProblem* prob, hipStream_t stream, const ReduceJob* jobs,
                                   int n_jobs, int rows) {
  if (!gemm_small_grouped_supported(dtype, n, prob)) {
    set_error("gemm_small_grouped: %d problems, or a shape, stride or pointer the kernel does not take", n);
    return false;
  }
  SmallGroup g;
  memset(&g, 0, sizeof(g));
  g.n = n;
  int64_t tiles64 = 0, tiles32 = 0;
  int K = prob[0].K;
  for (int i = 0; i < n; ++i) {
    const GemmProblem& q = prob[i];
    Epilogue ep;
    memset(&ep, 0, sizeof(ep));
    ep.acc_f32 = q.acc_f32;
    ep.ldc = q.ldc;
    g.p[i] = SmallProblem{q.A, q.B, ep, q.M, q.N, q.K, q.lda, q.ldb, 0, 0, vector_epilogue(dtype, ep)};
    tiles64 += (int64_t)ceil_div(q.M, 64) * ceil_div(q.N, 64);
    tiles32 += (int64_t)ceil_div(q.M, 32) * ceil_div(q.N, 32);
    K = min(K, q.K);
  }
  GroupSums sums;
  if (n_jobs > 0) {
    if (!make_reduce_batch(jobs, n_jobs, sums.batch)) return false;
    sums.rows = rows;
    sums.blocks = sums.batch.first64[n_jobs];
  }
  if (dtype == kF32 && !f32_few_tiles(tiles32, K)) return gemm_f32_grouped(g, n_jobs > 0 ? &sums : nullptr, stream);
  SmallForm f = small_form(dtype, tiles64, K);
  // a group of bf16 products does best with one wave per tile from 512 on:
  // width 512, 100 / 512 / 4000 rows 9.0 / 12.4 / 44.8 us against 10.7 / 14.5 / 49.9 with two
  if (dtype == kBF16 && tiles64 >= 512) f.waves = 1;
  return group_form(dtype, f, g, n_jobs > 0 ? &sums : nullptr, stream);
}

}  // namespace po
