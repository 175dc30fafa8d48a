// Column sums of several tensors (bias gradients, LayerNorm gain and shift gradients): the batch that the launches of
// elementwise.hip and the first blocks of a launch of weight-gradient products work through, and what such a block does.
#pragma once

#include "kernels.h"

namespace po {

struct ReduceBatch {
  ReduceJob job[kMaxReduceJobs];
  int first128[kMaxReduceJobs + 1];  // first 128-column block of job j on the partial kernel's grid.x
  int first64[kMaxReduceJobs + 1];   // first 64-column block of job j on the final kernel's grid.x
  int n_jobs;
};

// The batch of these jobs; false with error text if one of them is not complete.
bool make_reduce_batch(const ReduceJob* jobs, int n_jobs, ReduceBatch& b);
// Whether every job's rows are whole, aligned 16-byte vectors.
bool column_sums_vectors(int dtype, const ReduceJob* jobs, int n_jobs);

// Column sums of block `block` (as first64 numbers them, COLS = 32: twice as many halves of those), added to the job's results.  A
// lane takes one 16-byte vector of every SLOTS-th row.  The loads of AT_ONCE rows are in flight per lane (rows past the end are
// selected away and not branched round: a branch takes the loads with it); those rows are added in
// order, the sums of four such rounds in order, and those of these groups again: a fixed order whose chains are short however few
// slots there are, and a gain's last product is part of its addition.  The error against 64 bits is no larger than that of the sums
// over chunks of rows (0.93 to 1.01 of it).  One chain of rounds with trees of products in it was 5 % above with 16 slots and
// 600 rows, 13 % with 1536, and fp32 sums of 24 slots 5 % from 600 on.
// red: 2 COLS floats of LDS per wave.  Needs column_sums_vectors.
template <typename T, int THREADS, int COLS, int AT_ONCE>
__device__ __forceinline__ void column_sums_block(const ReduceBatch& b, int block, int rows, float* red) {
  constexpr int V = Vec16<T>::N, LPR = COLS / V, SLOTS = THREADS / LPR, WAVES = THREADS / kWave;
  constexpr int PER64 = 64 / COLS, GROUP = 4 * AT_ONCE * SLOTS;  // rows of a group of rounds
  int j = 0;
  while (j + 1 < b.n_jobs && block >= b.first64[j + 1] * PER64) ++j;
  const ReduceJob& job = b.job[j];
  const int n = job.n, col0 = (block - b.first64[j] * PER64) * COLS;
  const int cl = (int)threadIdx.x % LPR * V, slot = threadIdx.x / LPR;
  const bool inside = col0 + cl < n, ln = job.x != nullptr;
  const T* a = static_cast<const T*>(job.a) + col0 + cl;
  const T* x = static_cast<const T*>(job.x) + col0 + cl;
  float s0[V], s1[V];
#pragma unroll
  for (int i = 0; i < V; ++i) s0[i] = s1[i] = 0.f;
  if (inside && !ln) {
    for (int first = slot; first < rows; first += GROUP) {
      float g[V];
#pragma unroll
      for (int i = 0; i < V; ++i) g[i] = 0.f;
      for (int r0 = first; r0 < min(first + GROUP, rows); r0 += AT_ONCE * SLOTS) {
        Vec16<T> d[AT_ONCE];
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) d[u] = load16(a + (size_t)min(r0 + u * SLOTS, rows - 1) * n);
        float p[V];
#pragma unroll
        for (int i = 0; i < V; ++i) p[i] = 0.f;
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u)
#pragma unroll
          for (int i = 0; i < V; ++i) p[i] += r0 + u * SLOTS < rows ? to_f32(d[u].v[i]) : 0.f;
#pragma unroll
        for (int i = 0; i < V; ++i) g[i] += p[i];
      }
#pragma unroll
      for (int i = 0; i < V; ++i) s0[i] += g[i];
    }
  } else if (inside) {
    const float* stats = job.stats;
    for (int first = slot; first < rows; first += GROUP) {
      float g0[V], g1[V];
#pragma unroll
      for (int i = 0; i < V; ++i) g0[i] = g1[i] = 0.f;
      for (int r0 = first; r0 < min(first + GROUP, rows); r0 += AT_ONCE * SLOTS) {
        Vec16<T> d[AT_ONCE], xv[AT_ONCE];
        float mean[AT_ONCE], rstd[AT_ONCE];
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) {
          const size_t r = min(r0 + u * SLOTS, rows - 1);
          d[u] = load16(a + r * n);
          xv[u] = load16(x + r * n);
          mean[u] = stats[2 * r];
          rstd[u] = stats[2 * r + 1];
        }
        float p0[V], p1[V];
#pragma unroll
        for (int i = 0; i < V; ++i) p0[i] = p1[i] = 0.f;
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u)
#pragma unroll
          for (int i = 0; i < V; ++i) {
            // past the end 0 times the last row, which has put the NaN in already if that is one
            const float dv = r0 + u * SLOTS < rows ? to_f32(d[u].v[i]) : 0.f;
            p0[i] += dv * (to_f32(xv[u].v[i]) - mean[u]) * rstd[u];
            p1[i] += dv;
          }
#pragma unroll
        for (int i = 0; i < V; ++i) {
          g0[i] += p0[i];
          g1[i] += p1[i];
        }
      }
#pragma unroll
      for (int i = 0; i < V; ++i) {
        s0[i] += g0[i];
        s1[i] += g1[i];
      }
    }
  }
#pragma unroll
  for (int m = LPR; m < kWave; m <<= 1)
#pragma unroll
    for (int i = 0; i < V; ++i) {
      s0[i] += __shfl_xor(s0[i], m);
      if (ln) s1[i] += __shfl_xor(s1[i], m);
    }
  if ((threadIdx.x & 63) < LPR)
#pragma unroll
    for (int i = 0; i < V; ++i) {
      float* at = red + (threadIdx.x >> 6) * 2 * COLS + cl + i;
      at[0] = s0[i];
      at[COLS] = s1[i];
    }
  __syncthreads();
  for (int at = threadIdx.x; at < (ln ? 2 * COLS : COLS); at += THREADS) {
    const int c = at % COLS;
    if (col0 + c >= n) continue;
    float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < WAVES; ++w) part[w & 3] += red[w * 2 * COLS + at];
    (at >= COLS ? job.out1 : job.out0)[col0 + c] += (part[0] + part[1]) + (part[2] + part[3]);
  }
}

}  // namespace po
