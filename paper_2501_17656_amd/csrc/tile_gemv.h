// The wave program of the symmetric block products (coupling, projected close
// and stored near-field tiles), shared by the kernels that run it.
#pragma once

#include <hip/hip_runtime.h>

#include "device_common.h"

namespace h2mg {

template <typename Tv> __device__ inline Tv zero() { return Tv(0); }

__device__ inline int wave_id() {
  return __builtin_amdgcn_readfirstlane(int((blockIdx.x * blockDim.x + threadIdx.x) >> 6));
}

// One wave per task (row gid s, blocks [b0, b1)).  partial[task] = sum_b B_b x_{col b};
// colpart[slot of b] = B_b^T x_s for every off-diagonal block (slots are
// ordered by column, so the reduce reads each column's run contiguously).
// FULL: r == 8T (no padding, no guards).  Each iteration requests its tile
// first, then the coefficients of its column (the next column index is
// prefetched by a scalar load), so one tile is in flight per wave while the
// previous is consumed.  Every tile is read once per launch, with
// non-temporal loads (measured faster than ordinary loads for FP64, FP32 and
// BF16 tiles alike on the same machine and run).  PARTS: the rows of a sub-tile
// are read in that many turns, for kernels that must leave more registers to
// others (a 64 x 64 FP64 tile at once takes 128 of them).
template <int T, bool FULL, int PARTS, typename Tb, typename Tv>
__device__ __forceinline__ void bsr_gemv_wave(int wave, const int* __restrict__ tasks, int ntasks,
                                              const Tb* __restrict__ blk,
                                              const int* __restrict__ blk_col,
                                              const int* __restrict__ blk_slot,
                                              const Tv* __restrict__ x, Tv* __restrict__ partial,
                                              Tv* __restrict__ colpart, int r, int A) {
  constexpr int TP = T / PARTS;
  if (wave >= ntasks) return;
  const int lane = threadIdx.x & 63;
  const int a = lane >> 3, b = lane & 7;
  const int row = tasks[3 * wave], b0 = tasks[3 * wave + 1], b1 = tasks[3 * wave + 2];
  const int rr = FULL ? 8 * T : r;
  Tv xs[T], acc[T];
#pragma unroll
  for (int u = 0; u < T; ++u) {
    const int i = a * T + u;
    xs[u] = (FULL || i < rr) ? x[int64_t(row) * rr + i] : zero<Tv>();
    acc[u] = zero<Tv>();
  }
  int col = blk_col[b0];
  for (int bi = b0; bi < b1; ++bi) {
    Tv B[TP * T];
    const Tb* tile = blk + int64_t(bi) * tile_elems(T);
    load_subtile<T, Tb, Tv, true, PARTS>(tile, lane, A, B);
    const int col_next = bi + 1 < b1 ? blk_col[bi + 1] : col;
    Tv xt[T], z[T];
#pragma unroll
    for (int v = 0; v < T; ++v) {
      const int j = b * T + v;
      xt[v] = (FULL || j < rr) ? x[int64_t(col) * rr + j] : zero<Tv>();
      z[v] = zero<Tv>();
    }
#pragma unroll
    for (int q = 0; q < PARTS; ++q) {
      if (q > 0) {
        __builtin_amdgcn_sched_barrier(0);       // the parts take turns in B's registers
        load_subtile<T, Tb, Tv, true, PARTS>(tile, lane, A, B, q);
      }
#pragma unroll
      for (int u = 0; u < TP; ++u)
#pragma unroll
        for (int v = 0; v < T; ++v) {
          acc[q * TP + u] += B[u * T + v] * xt[v];
          z[v] += B[u * T + v] * xs[q * TP + u];
        }
      if constexpr (PARTS > 1) {
        // both sums are formed here, not where they are used: that would keep
        // every part in registers
#pragma unroll
        for (int v = 0; v < T; ++v) asm volatile("" : "+v"(z[v]));
#pragma unroll
        for (int u = 0; u < TP; ++u) asm volatile("" : "+v"(acc[q * TP + u]));
      }
    }
    if (col != row) {
      const Tv zs = transpose_reduce_a<T, Tv>(z, a);
      const int v = reduced_index<T>(a);
      const int j = b * T + v;
      if ((T == 8 || (a & ((8 / T) - 1)) == 0) && (FULL || j < rr))
        colpart[int64_t(blk_slot[bi]) * rr + j] = zs;
    }
    col = col_next;
  }
#pragma unroll
  for (int u = 0; u < T; ++u) {
    Tv s = acc[u];
    s += shfl_xor(s, 1);
    s += shfl_xor(s, 2);
    s += shfl_xor(s, 4);
    acc[u] = s;
  }
  if (b == 0) {
#pragma unroll
    for (int u = 0; u < T; ++u) {
      const int i = a * T + u;
      if (FULL || i < rr) partial[int64_t(wave) * rr + i] = acc[u];
    }
  }
}

}  // namespace h2mg
