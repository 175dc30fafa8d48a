// GEMM on the matrix cores for any M, N, K and for fp32 as well as bf16: the kernel of fp32 stages, of short or narrow
// operands whose 128 x 128 tiles would leave most of the chip idle, and of everything that is no multiple of a tile.
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
// banks.
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

  // p: the operand; ld in elements; row0: first row of the tile (of `rows`); chunk: this wave's first chunk of K.
  __device__ __forceinline__ void init(const T* p, int ld, int row0, int rows, int K, int chunk, int chunk_step, int lane) {
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
      int byte = u * 1024 + lane * 16;
      if (!KMAJOR) {
        int row = byte >> 7, c = ((byte >> 4) & 7) ^ (row & 7);
        voff[u] = (unsigned)row * (unsigned)ld * E + c * 16;
      } else {
        int k = byte / ROW_BYTES, c = piece_of((byte % ROW_BYTES) >> 4, k);
        voff[u] = (unsigned)k * (unsigned)ld * E + c * 16;
      }
    }
    int64_t first = KMAJOR ? (int64_t)chunk * KU * ld + row0 : (int64_t)row0 * ld + (int64_t)chunk * KU;
    int64_t end = KMAJOR ? (int64_t)(K - 1) * ld + rows : (int64_t)(rows - 1) * ld + K;
    base = reinterpret_cast<const char*>(p) + first * E;
    left = (end - first) * E;
    step = (int64_t)chunk_step * (KMAJOR ? (int64_t)KU * ld * E : 128);
  }
  // Requests the chunk at `base` into LDS at `lds`; k_left: how many k the chunk has (>= KU: all of them).
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

template <typename T, int TM, int TN, int KG, bool TA, bool TB>
__device__ __forceinline__ void small_tile(const SmallProblem& p, int tile, char* smem) {
  constexpr int BM = 32 * TM, BN = 32 * TN, KU = MfmaOf<T>::KU;
  using OpA = Operand<T, BM, TA>;
  using OpB = Operand<T, BN, TB>;
  constexpr int STAGE = OpA::BYTES + OpB::BYTES, LOADS = OpA::LOADS + OpB::LOADS;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // tiles in groups of eight rows, so that a run of them is compact in both dimensions
  const int M = p.M, N = p.N, K = p.K;
  const int tiles_m = (M + BM - 1) / BM, first = tile / (8 * p.tiles_n) * 8, rows = min(tiles_m - first, 8);
  const int at = tile - first * p.tiles_n;
  const int m0 = (first + at % rows) * BM, n0 = at / rows * BN;

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

// Block ids equal modulo 8 share an XCD: each XCD gets a run of neighbouring tiles (and their operands its L2).
__device__ __forceinline__ int tile_of_block() {
  const int n = gridDim.x, pid = blockIdx.x;
  return n % 8 == 0 ? (pid % 8) * (n / 8) + pid / 8 : pid;
}

template <typename T, int TM, int TN, int KG, bool TA, bool TB>
__global__ __launch_bounds__(64 * KG) void gemm_small_kernel(SmallProblem p) {
  extern __shared__ __align__(16) char smem[];
  small_tile<T, TM, TN, KG, TA, TB>(p, tile_of_block(), smem);
}

// The four weight-gradient products of a layer in one launch: the tiles of all of them one product after the other.
constexpr int kMaxSmallGroup = 4;
struct SmallGroup {
  SmallProblem p[kMaxSmallGroup];
  int n;
};
template <typename T, int TM, int TN, int KG>
__global__ __launch_bounds__(64 * KG) void gemm_small_grouped_kernel(SmallGroup g) {
  extern __shared__ __align__(16) char smem[];
  const int lin = tile_of_block();
  SmallProblem p = g.p[0];  // constant indices only: a run-time index would send the arguments through memory
#pragma unroll
  for (int i = 1; i < kMaxSmallGroup; ++i)
    if (i < g.n && lin >= g.p[i].first_tile) p = g.p[i];
  small_tile<T, TM, TN, KG, true, true>(p, lin - p.first_tile, smem);
}

// ---- host side -------------------------------------------------------------------------------------------------
// Waves of a block and its tile.  Times in us of one launch with warm operands, forms 32x32 with 8 and 4 waves, 64x64
// with 4, 2 and 1 waves:
//   bf16  512 x  512, K  512:  3.8  3.6   5.0   5.8   8.6        bf16  512 x 1536, K  512:  8.9  6.3  5.1  5.9  8.7
//   bf16  512 x  512, K 2048:  7.5  6.1   9.0  12.8  21.8        bf16 1024 x 1024, K 1024: 13.4  9.6  6.7  8.3 13.3
//   bf16  100 x 2048, K 8192: 19.0 19.4  25.3  39.9  73.7        bf16  100 x 8192, K 2048: 22.2 17.7 10.7 13.3 22.0
//   bf16 2048 x 2048, K  100: 30.0 16.3  14.6  11.2   9.8        bf16 1733 x 6144, K 2048:  207  140   86   76   72
//   fp32  128 x  256, K 1024:  8.0  8.3  21.0  37.8  72.2        fp32 1024 x 1024, K 1024: 28.4 25.6 22.3 38.0 71.9
//   fp32 1024 x 1024, K 4096: 90.3 95.9  75.3   140   272        fp32 4096 x 1024, K 1024:  116   93   88  134   81
// A 32 x 32 tile halves what an operand byte is used for but makes four times as many blocks: it wins while 64 x 64
// tiles leave half of the CUs without one.  From there on more waves per tile shorten its chain of chunks, as long as
// every wave has a few chunks and the chip is not full anyway: fp32, whose MFMAs take eight times as long per byte,
// always has four; bf16 has as many as keep four waves on every CU.
struct SmallForm {
  int edge, waves;
};
static SmallForm small_form(int dtype, int64_t tiles64, int K) {
  const int chunks = ceil_div(K, dtype == kF32 ? 32 : 64);
  if (tiles64 < 128) return {32, dtype == kF32 && chunks >= 16 ? 8 : 4};
  int waves = tiles64 < 512 ? 4 : tiles64 < 1024 ? 2 : 1;
  if (dtype == kF32) waves = tiles64 < 1024 || chunks > 8 ? 4 : 1;
  while (waves > 1 && chunks < 2 * waves) waves /= 2;
  return {64, waves};
}

static bool vector_epilogue(int dtype, const Epilogue& ep) {
  const int v = dtype == kF32 ? 4 : 8;
  return ep.ldc % v == 0 && ((uintptr_t)ep.bias | (uintptr_t)ep.residual | (uintptr_t)ep.out | (uintptr_t)ep.gelu_out |
                             (uintptr_t)ep.gelu_u | (uintptr_t)ep.acc_f32) % 16 == 0;
}

bool gemm_small_supported(int dtype, int trans_a, int trans_b, int M, int N, int K, const void* A, int lda,
                          const void* B, int ldb) {
  const int v = dtype == kF32 ? 4 : 8;  // elements of a 16-byte load
  // rows of both operands are whole 16-byte pieces; a lane's offset (up to 64 rows) fits 32 bits
  const int64_t limit = (int64_t)1 << 31;
  return M > 0 && N > 0 && K > 0 && lda % v == 0 && ldb % v == 0 && (trans_a ? M : K) % v == 0 &&
         (trans_b ? K : N) % v == 0 && ((uintptr_t)A | (uintptr_t)B) % 16 == 0 && (int64_t)lda * 64 * 4 < limit &&
         (int64_t)ldb * 64 * 4 < limit;
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

template <typename T>
static bool launch_form(SmallForm f, int ta, int tb, SmallProblem& p, hipStream_t stream) {
  if (f.edge == 32) {
    if constexpr (sizeof(T) == 4)  // small_form gives fp32 alone eight
      if (f.waves == 8) return launch_trans<T, 1, 1, 8>(ta, tb, p, stream);
    return launch_trans<T, 1, 1, 4>(ta, tb, p, stream);
  }
  if (f.waves == 4) return launch_trans<T, 2, 2, 4>(ta, tb, p, stream);
  if (f.waves == 2) return launch_trans<T, 2, 2, 2>(ta, tb, p, stream);
  return launch_trans<T, 2, 2, 1>(ta, tb, p, stream);
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
  SmallForm f = small_form(dtype, (int64_t)ceil_div(M, 64) * ceil_div(N, 64), K);
  return dtype == kF32 ? launch_form<float>(f, ta, tb, p, stream) : launch_form<bf16>(f, ta, tb, p, stream);
}

template <typename T, int TM, int TN, int KG>
static bool launch_group(SmallGroup& g, hipStream_t stream) {
  constexpr int smem = KG * 2 * 32 * (TM + TN) * 128;
  auto kern = gemm_small_grouped_kernel<T, TM, TN, KG>;
  static LdsLimit lds;
  if (!lds.allow(kern, smem)) return false;
  int total = 0;
  for (int i = 0; i < g.n; ++i) {
    g.p[i].tiles_n = ceil_div(g.p[i].N, 32 * TN);
    g.p[i].first_tile = total;
    total += ceil_div(g.p[i].M, 32 * TM) * g.p[i].tiles_n;
  }
  kern<<<total, 64 * KG, smem, stream>>>(g);
  return launch_ok("gemm_small_grouped_kernel");
}

template <typename T>
static bool group_form(SmallForm f, SmallGroup& g, hipStream_t stream) {
  if (f.edge == 32) {
    if constexpr (sizeof(T) == 4)
      if (f.waves == 8) return launch_group<T, 1, 1, 8>(g, stream);
    return launch_group<T, 1, 1, 4>(g, stream);
  }
  if (f.waves == 4) return launch_group<T, 2, 2, 4>(g, stream);
  if (f.waves == 2) return launch_group<T, 2, 2, 2>(g, stream);
  return launch_group<T, 2, 2, 1>(g, stream);
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

bool gemm_small_grouped_accumulate(int dtype, int n, const GemmProblem* prob, hipStream_t stream) {
  if (!gemm_small_grouped_supported(dtype, n, prob)) {
    set_error("gemm_small_grouped: %d problems, or a shape, stride or pointer the kernel does not take", n);
    return false;
  }
  SmallGroup g;
  memset(&g, 0, sizeof(g));
  g.n = n;
  int64_t tiles64 = 0;
  int K = prob[0].K;
  for (int i = 0; i < n; ++i) {
    const GemmProblem& q = prob[i];
    Epilogue ep;
    memset(&ep, 0, sizeof(ep));
    ep.acc_f32 = q.acc_f32;
    ep.ldc = q.ldc;
    g.p[i] = SmallProblem{q.A, q.B, ep, q.M, q.N, q.K, q.lda, q.ldb, 0, 0, vector_epilogue(dtype, ep)};
    tiles64 += (int64_t)ceil_div(q.M, 64) * ceil_div(q.N, 64);
    K = min(K, q.K);
  }
  SmallForm f = small_form(dtype, tiles64, K);
  // a group of bf16 products does best with one wave per tile from 512 on:
  // width 512, 100 / 512 / 4000 rows 9.0 / 12.4 / 44.8 us against 10.7 / 14.5 / 49.9 with two
  if (dtype == kBF16 && tiles64 >= 512) f.waves = 1;
  return dtype == kF32 ? group_form<float>(f, g, stream) : group_form<bf16>(f, g, stream);
}

}  // namespace po
