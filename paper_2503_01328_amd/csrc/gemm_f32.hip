// fp32 GEMM on v_mfma_f32_32x32x2_f32 (full fp32 products and sums, 256 flop/clk/CU: 157 TFLOP/s at 2.4 GHz) for results
// of more tiles than one round of 32 x 32 ones; smaller ones have gemm_small.hip.
//
// An MFMA takes 64 cycles, so operands are cheap to supply and what decides is that no SIMD's matrix core waits.  The waves
// of a block share each chunk of K (32 k, 128 bytes of a row) through a ring of NST LDS stages.  A wave that issues a tile load
// is held until the memory pipeline has taken it, so two waves of the block do nothing else, one per operand (one for both
// cannot feed 64 x 64 tiles: a chunk's 16 loads take it longer than the chunk's MFMAs); the computing waves only read
// fragments, each behind an MFMA of the step before its own, and multiply.  The one barrier per chunk stands where the last of the
// chunk's fragments are in registers and a quarter of its MFMAs is still to come.  Two or three blocks share a CU: one's
// first loads and last stores run under the other's MFMAs.  LDS has room for them (48 to 72 KB a block); the registers have up to
// 80 a wave, since the first SIMD takes two of a block's six waves (three of ten): four accumulators kept to the end
// instead of two and a sum (90 registers) cost 5 to 15 % wherever a CU gets more than two tiles.
//
// A block: WK groups of WM x WN computing waves, a wave one tile of 32 x 32.  Group g owns every WK-th chunk; the
// groups' partial tiles are added in group order through LDS (always the same order: deterministic).  Chunks past K and
// rows past M or N read as zero (the buffer descriptors end with the operand), the epilogue stores only what is inside.
//
// Rounding: every sum is formed in at least four chains of a quarter of K (eight of an eighth in 32 x 64 tiles).  Against 64 bits,
// normal operands, K 512 / 1024 / 8192: 2.1e-7, 2.9e-7, 8.1e-7; one chain has twice, two have 1.4 times that, and with operands of one
// sign 3.7 and 1.9 times.
//
// Measured against tiles of 64 x 64 whose four waves each took every fourth chunk of K and loaded it themselves, the same
// chains (us): 1024 x 4096, K 1024 81 -> 71 (121 TFLOP/s); 2048 x 2048, K 8192 552 -> 502 (137); 777 x 640, K 2560 46 -> 25;
// 512 x 2560, K 5120 174 -> 124; 4096 x 1536, K 512 71 -> 54.  What is left: the barrier (a SIMD's pipe runs dry while the last
// wave arrives) and the last, partly filled round of tiles.
#include <string.h>

#include "gemm_tile.h"

namespace po {

template <int WM_, int WN_, int WK_, int NST_>
struct F32Form {
  static constexpr int WM = WM_, WN = WN_, WK = WK_, NST = NST_;
  static constexpr int BM = 32 * WM, BN = 32 * WN, GW = WM * WN, WAVES = GW * WK;  // computing waves
  static constexpr int THREADS = 64 * (WAVES + 2);
  static constexpr int STAGE = (BM + BN) * 128, LD = BN + 4;
  static constexpr int RING = NST * STAGE > BM * LD * 4 ? NST * STAGE : BM * LD * 4;  // of a group; later its partial tile
  static constexpr int SMEM = WK * RING;
};

template <typename Form, bool TA, bool TB>
__device__ __forceinline__ void f32_tile(const SmallProblem& p, int tile, char* smem) {
  constexpr int WN = Form::WN, WK = Form::WK, NST = Form::NST;
  constexpr int BM = Form::BM, BN = Form::BN, GW = Form::GW, KU = MfmaOf<float>::KU;
  static_assert(BM <= kMaxSmallRows && BN <= kMaxSmallRows, "gemm_small_supported bounds a lane's offset");
  using OpA = Operand<float, BM, TA>;
  using OpB = Operand<float, BN, TB>;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int group = wave / GW, w = wave % GW, wm = w / WN, wn = w % WN;
  const int M = p.M, N = p.N, K = p.K;
  int m0, n0;
  place_of_tile(tile, (M + BM - 1) / BM, p.tiles_n, m0, n0);
  m0 *= BM;
  n0 *= BN;

  const int chunks = ((K + KU - 1) / KU + WK - 1) / WK;  // of every group; the last ones may be empty
  // Four chains of additions: even and odd pairs of k, the first and the second half of the chunks.
  f32x16 acc[2], first_half;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[0][e] = acc[1][e] = 0.f;
  // Loader waves: one for A, one for B.
  auto loader = [&](auto op, const float* ptr, int ld, int row0, int rows, int offset) {
    using Op = decltype(op);
    constexpr int LOADS = WK * Op::LOADS;  // of a chunk of every group
    Op x[WK];
#pragma unroll
    for (int g = 0; g < WK; ++g) x[g].init(ptr, ld, row0, rows, K, g, WK, lane);
    const unsigned ring = __builtin_amdgcn_readfirstlane((int)lds_byte(smem)) + offset;
    int k_left = K;
    auto issue = [&](unsigned stage) {
#pragma unroll
      for (int g = 0; g < WK; ++g) x[g].issue(ring + g * Form::RING + stage, k_left - g * KU, lane);
      k_left -= WK * KU;
    };
#pragma unroll
    for (int i = 0; i < NST; ++i) issue(i * Form::STAGE);
    wait_loads<(LOADS * (NST - 1) < 63 ? LOADS * (NST - 1) : 63)>();
    asm volatile("s_barrier" ::: "memory");
    unsigned stage = 0;
    for (int t = 0; t < chunks; ++t) {
      wait_loads<(LOADS * (NST - 2) < 63 ? LOADS * (NST - 2) : 63)>();
      asm volatile("s_barrier" ::: "memory");
      issue(stage);
      stage = stage + Form::STAGE == NST * Form::STAGE ? 0 : stage + Form::STAGE;
    }
    wait_loads<0>();  // the empty chunks behind the last one write zeros into the ring
  };
  if (wave == Form::WAVES) {
    loader(OpA(), static_cast<const float*>(p.A), p.lda, m0, M, 0);
  } else if (wave == Form::WAVES + 1) {
    loader(OpB(), static_cast<const float*>(p.B), p.ldb, n0, N, OpA::BYTES);
  } else {
    const char* ring = smem + group * Form::RING;
    f32x4 fa[2], fb[2];
    auto read_a = [&](unsigned stage, int kk, int buf) {
      fa[buf] = fragment<BM, TA>((const float*)nullptr, ring + stage, 32 * wm, kk, lane);
    };
    auto read_b = [&](unsigned stage, int kk, int buf) {
      fb[buf] = fragment<BN, TB>((const float*)nullptr, ring + stage + OpA::BYTES, 32 * wn, kk, lane);
    };
    asm volatile("s_barrier" ::: "memory");
    unsigned stage = 0;
    read_a(0, 0, 0);
    read_b(0, 0, 0);
    auto multiply_chunks = [&](int n) __attribute__((always_inline)) {
      for (int t = 0; t < n; ++t) {
        const unsigned next = stage + Form::STAGE == NST * Form::STAGE ? 0 : stage + Form::STAGE;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          if (kk == 3) {  // this wave has the last fragments of the chunk; when all have them the stage is free
            wait_lds_reads();
            asm volatile("s_barrier" ::: "memory");
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            acc[e & 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[kk & 1][e], fa[kk & 1][e], acc[e & 1], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (e == 0) read_a(kk < 3 ? stage : next, (kk + 1) & 3, (kk + 1) & 1);
            if (e == 1) read_b(kk < 3 ? stage : next, (kk + 1) & 3, (kk + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        stage = next;
      }
    };
    const int half = chunks >= 4 ? chunks / 2 : 0;
    multiply_chunks(half);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      first_half[e] = acc[0][e] + acc[1][e];
      asm volatile("" : "+v"(first_half[e]));  // here: left to itself the compiler keeps all four chains to the end
      acc[0][e] = acc[1][e] = 0.f;
    }
    multiply_chunks(chunks - half);
    wait_lds_reads();
  }
  __syncthreads();

  constexpr int LD = Form::LD;
  float* part = reinterpret_cast<float*>(smem + group * Form::RING);
  if (wave < Form::WAVES) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = first_half[4 * q + e] + (acc[0][4 * q + e] + acc[1][4 * q + e]);
      *reinterpret_cast<f32x4*>(part + (32 * wm + (lane & 31)) * LD + 32 * wn + 8 * q + 4 * (lane >> 5)) = v;
    }
  }
  __syncthreads();
  constexpr int PER_ROW = BN / 4;
#pragma unroll 4
  for (int piece = threadIdx.x; piece < BM * PER_ROW; piece += Form::THREADS) {
    int r = piece / PER_ROW, c = piece % PER_ROW * 4;
    if (m0 + r >= M || n0 + c >= N) continue;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int g = 0; g < WK; ++g) {
      f32x4 x = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(smem + g * Form::RING) + r * LD + c);
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] += x[k];
    }
    if (p.vec && n0 + c + 4 <= N) {
      epilogue_vector<float>(p.ep, m0 + r, n0 + c, v);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (n0 + c + i < N) epilogue_store<float>(p.ep, m0 + r, n0 + c + i, v[i]);
    }
  }
}

// The tile of a block of a grid of gemm_f32_grid; of a second dimension the last blocks have none.
__device__ __forceinline__ int tile_of_f32_block() {
  return gridDim.y == 1 ? tile_of_block() : (int)(blockIdx.y * gridDim.x + blockIdx.x);
}

template <typename Form, bool TA, bool TB>
__global__ __launch_bounds__(Form::THREADS) void gemm_f32_kernel(SmallProblem p) {
  extern __shared__ __align__(16) char smem[];
  const int tile = tile_of_f32_block();
  if (tile < (p.M + Form::BM - 1) / Form::BM * p.tiles_n) f32_tile<Form, TA, TB>(p, tile, smem);
}

template <typename Form>
__device__ __forceinline__ void f32_group_tile(const SmallGroup& g, int lin, char* smem) {
  if (lin >= g.tiles) return;
  SmallProblem p = g.p[0];  // constant indices only: a run-time index would send the arguments through memory
#pragma unroll
  for (int i = 1; i < kMaxSmallGroup; ++i)
    if (i < g.n && lin >= g.p[i].first_tile) p = g.p[i];
  f32_tile<Form, true, true>(p, lin - p.first_tile, smem);
}
template <typename Form>
__global__ __launch_bounds__(Form::THREADS) void gemm_f32_grouped_kernel(SmallGroup g) {
  extern __shared__ __align__(16) char smem[];
  f32_group_tile<Form>(g, tile_of_f32_block(), smem);
}
// And its column sums, in blocks of their own before the others, which hide them (a grid of one dimension).
template <typename Form>
__global__ __launch_bounds__(Form::THREADS) void gemm_f32_with_sums_kernel(SmallGroup g, GroupSums sums) {
  extern __shared__ __align__(16) char smem[];
  if ((int)blockIdx.x < sums.blocks)
    column_sums_block<float, Form::THREADS, 64, 4>(sums.batch, blockIdx.x, sums.rows, reinterpret_cast<float*>(smem));
  else
    f32_group_tile<Form>(g, tile_of_block(sums.blocks), smem);
}

// A dimension of a grid ends at 2^32 threads.
dim3 gemm_f32_grid(int64_t tiles, int threads) {
  const unsigned y = (unsigned)ceil_div64(tiles * threads, (int64_t)1 << 31);
  return dim3((unsigned)ceil_div64(tiles, y), y);
}
template <typename Form, bool TA, bool TB>
static bool launch_one(SmallProblem& p, hipStream_t stream) {
  auto kern = gemm_f32_kernel<Form, TA, TB>;
  static LdsLimit lds;  // per instantiation
  if (!lds.allow(kern, Form::SMEM)) return false;
  p.tiles_n = ceil_div(p.N, Form::BN);
  kern<<<gemm_f32_grid(ceil_div(p.M, Form::BM) * p.tiles_n, Form::THREADS), Form::THREADS, Form::SMEM, stream>>>(p);
  return launch_ok("gemm_f32_kernel");
}
template <typename Form>
static bool launch_trans(int ta, int tb, SmallProblem& p, hipStream_t stream) {
  // kernel flag TB means "B is n-contiguous", i.e. trans_b == 0
  if (!ta && !tb) return launch_one<Form, false, true>(p, stream);
  if (!ta && tb) return launch_one<Form, false, false>(p, stream);
  if (ta && !tb) return launch_one<Form, true, true>(p, stream);
  return launch_one<Form, true, false>(p, stream);
}
template <typename Form>
static bool launch_group(SmallGroup& g, const GroupSums* sums, hipStream_t stream) {
  int total = 0;
  for (int i = 0; i < g.n; ++i) {
    g.p[i].tiles_n = ceil_div(g.p[i].N, Form::BN);
    g.p[i].first_tile = total;
    total += ceil_div(g.p[i].M, Form::BM) * g.p[i].tiles_n;
  }
  g.tiles = total;
  if (sums) {
    auto kern = gemm_f32_with_sums_kernel<Form>;
    static LdsLimit lds;
    if (!lds.allow(kern, Form::SMEM)) return false;
    kern<<<total + sums->blocks, Form::THREADS, Form::SMEM, stream>>>(g, *sums);
    return launch_ok("gemm_f32_with_sums_kernel");
  }
  auto kern = gemm_f32_grouped_kernel<Form>;
  static LdsLimit lds;
  if (!lds.allow(kern, Form::SMEM)) return false;
  kern<<<gemm_f32_grid(total, Form::THREADS), Form::THREADS, Form::SMEM, stream>>>(g);
  return launch_ok("gemm_f32_grouped_kernel");
}

// ---- which tile -----------------------------------------------------------------------------------------------------
// Form 0: 32 x 64, two groups of two waves; 1: 64 x 64, four waves; 2: 128 x 64, eight waves.  Small tiles fill the last
// round better, big ones read an operand less often, and the last also has fewer blocks to start and end.  A launch takes as long
// as its fullest CU: rounds of tiles times (start + per chunk of K), in us, fitted to 100 products of 32 to 6000 rows, columns and
// k: 6 % off on average, 26 % at most (the least launches); the choice is within 0.5 % of the best form on average and 9 % at most.
// Forms 0, 1 and 2, us:
//   1024 x 1024, K 1024: 24.0 23.2 36.0    1024 x 4096, K 1024: 84.5 79.0 77.2    780 x 640, K 2560: 26.7 43.9 79.9
//   1500 x 1536, K 1536: 68.8 73.5 93.9    4608 x 1536, K 1500:  192  189  208    4096 x 512, K 512: 23.0 20.7 20.5
//   2004 x 2936, K  788:  110 90.2 78.8    4096 x 4096, K 4096: 1060 1010 1059    2072 x 4480, K 472: 108 91.5 96.0
using Form32x64 = F32Form<1, 2, 2, 3>;
using Form64x64 = F32Form<2, 2, 1, 3>;
using Form128x64 = F32Form<4, 2, 1, 2>;
static double round_time(int form, int64_t tiles, int K) {
  static const double start[3] = {1.34, 1.19, 2.11}, chunk[3] = {0.517, 0.493, 0.936}, last[3] = {0.60, 0.63, 1.0};
  const int chunks = form == 0 ? ceil_div(ceil_div(K, 32), 2) : ceil_div(K, 32);
  // few rounds: whole ones; many: the blocks of a CU no longer end together
  const double rounds = tiles <= 768 ? (double)ceil_div64(tiles, 256) : (double)tiles / 256 + last[form];
  return rounds * (start[form] + chunk[form] * chunks);
}
static void count_tiles(int M, int N, int64_t* tiles) {
  tiles[0] += (int64_t)ceil_div(M, 32) * ceil_div(N, 64);
  tiles[1] += (int64_t)ceil_div(M, 64) * ceil_div(N, 64);
  tiles[2] += (int64_t)ceil_div(M, 128) * ceil_div(N, 64);
}
// The form of one launch for n products (the smallest K counts).
int gemm_f32_form(int n, const int* M, const int* N, int K) {
  int64_t tiles[3] = {0, 0, 0};
  for (int i = 0; i < n; ++i) count_tiles(M[i], N[i], tiles);
  int best = 0;
  for (int f = 1; f < 3; ++f)
    if (round_time(f, tiles[f], K) < round_time(best, tiles[best], K)) best = f;
  return best;
}

bool gemm_f32(int ta, int tb, SmallProblem& p, hipStream_t stream) {
  switch (gemm_f32_form(1, &p.M, &p.N, p.K)) {
    case 0: return launch_trans<Form32x64>(ta, tb, p, stream);
    case 1: return launch_trans<Form64x64>(ta, tb, p, stream);
    default: return launch_trans<Form128x64>(ta, tb, p, stream);
  }
}

bool gemm_f32_grouped(SmallGroup& g, const GroupSums* sums, hipStream_t stream) {
  int M[kMaxSmallGroup], N[kMaxSmallGroup], K = g.p[0].K;
  for (int i = 0; i < g.n; ++i) {
    M[i] = g.p[i].M;
    N[i] = g.p[i].N;
    K = min(K, g.p[i].K);
  }
  switch (gemm_f32_form(g.n, M, N, K)) {
    case 0: return launch_group<Form32x64>(g, sums, stream);
    case 1: return launch_group<Form64x64>(g, sums, stream);
    default: return launch_group<Form128x64>(g, sums, stream);
  }
}

}  // namespace po
