// The evaluated near field of the H2 matvec (Section 3.1: y = D x on the
// close leaf pairs), one vector, the entries formed from the points in every
// product.
//
// FP64 vector issue bounds it (32 operations an entry), so what counts
// is that no entry is formed for padding and that nothing else is issued.
//   * One wave per task: a row leaf s and a run of its close pairs (s <= t),
//     in chunks of up to 64 rows.  No LDS and no barrier, so the waves of a
//     workgroup are independent.
//   * Lane (ti, tj) = (lane % 8, lane / 8) holds the points of rows ti + 8u,
//     u < U, in registers and walks the columns tj + 8v, the next column's
//     point on its way while the current one is used; each entry feeds the
//     row sum (kept over the whole task) and the column sum.  Rows and columns
//     are padded to multiples of 8 only: U is one of 1 .. 8, chosen per chunk
//     among loops unrolled for each.  The earlier form, 256 threads on
//     128 x 128 tiles, formed 16384 entries also for a pair of 49-point
//     leaves.
//   * A column sum over the 8 lanes of a column takes three DPP steps per 8 U
//     entries; eight columns are collected and written as one 64-word run.
// Measured, one FP64 pass (128 x 128 tiles / now): 2270 / 420 us on 50000 points
// of a Gaussian mixture (leaves of 49), 1059 / 125 us on a 300 x 300 grid (leaves
// of 44), 40 / 14 us on 4096 points, 3073 / 1790 us (with the cheaper entries) on
// 131072 points with full leaves, where three waves per SIMD issue an FP64
// operation every 5.3 cycles (eight would reach 4.5).
#include <hip/hip_runtime.h>

#include <stdexcept>
#include <string>

#include "h2_impl.h"
#include "tile_gemv.h"

namespace h2mg {

namespace {

void check_launch(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) throw std::runtime_error(std::string(what) + ": " + hipGetErrorString(e));
}

// v plus its value in the lane that the DPP control pairs it with.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
  return v + __hiloint2double(hi, lo);
}
// Sum over the 8 lanes that share lane / 8, in every one of them: lane ^ 1,
// lane ^ 2 (quad permutations), then the other quad (half-row mirror).
template <typename Tv>
__device__ __forceinline__ Tv sum8(Tv v) {
  return dpp_add<0x141>(dpp_add<0x4E>(dpp_add<0xB1>(v)));
}

template <typename Tv>
struct NearIn {
  const int* pair_col;
  const int* pair_slot;
  const int* leaf_off;
  const double* pts;
  const double* scale;
  const Tv* x;
  Tv* partial;
  Tv* colpart;
  KernelParams kp;
  int ld, nsplit;
};

// Rows [rt, rt + nrow) of leaf sl (U >= nrow / 8) against the pairs [p0, p1).
// first: this wave has not written these pairs' column sums yet.  MINED: the
// squared distance starts at MIN_R2 (its first addition is an FMA, so that
// costs nothing) and the kernel need not bound its arguments.  NORMAL: no FP32
// entry is subnormal.
template <int U, int DIM, bool MINED, bool NORMAL, typename Tv, int KIND, int DERIV>
__device__ __forceinline__ void near_rows(const NearIn<Tv>& A, int task, int part, int sl, int p0, int p1, int rt,
                                          int nrow, bool first) {
  const int lane = threadIdx.x & 63;
  const int ti = lane & 7, tj = lane >> 3;
  const int s0 = A.leaf_off[sl] + rt;
  double pi[U][DIM];
  Tv xi[U], racc[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) racc[u] = Tv(0);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = ti + 8 * u;
    const int64_t gi = s0 + min(i, nrow - 1);
#pragma unroll
    for (int a = 0; a < DIM; ++a) pi[u][a] = A.pts[gi * DIM + a];
    xi[u] = i < nrow ? (A.scale ? Tv(A.scale[gi]) * A.x[gi] : A.x[gi]) : Tv(0);
  }
  double pn[DIM];
  Tv xn;
  auto load = [&](int t0, int nt, int v) {
    const int j = tj + 8 * v;
    const int64_t gj = t0 + min(j, nt - 1);
#pragma unroll
    for (int a = 0; a < DIM; ++a) pn[a] = A.pts[gj * DIM + a];
    xn = A.scale ? Tv(A.scale[gj]) * A.x[gj] : A.x[gj];
    if (j >= nt) xn = Tv(0);
  };
  int tl = A.pair_col[p0];
  int t0 = A.leaf_off[tl], nt = A.leaf_off[tl + 1] - t0;
  load(t0, nt, 0);
  const KernelConst<Tv> kc(A.kp);
  for (int p = p0; p < p1; ++p) {
    const int slot = A.pair_slot[p];
    Tv* dst = slot < 0 ? nullptr : A.colpart + (int64_t(slot) * A.nsplit + part) * A.ld;
    const int nv = (nt + 7) >> 3;
    const int tc0 = t0, ntc = nt;
    if (p + 1 < p1) {
      tl = A.pair_col[p + 1];
      t0 = A.leaf_off[tl];
      nt = A.leaf_off[tl + 1] - t0;
    }
    Tv keep = Tv(0), old = Tv(0);
    for (int v = 0; v < nv; ++v) {
      double pj[DIM];
#pragma unroll
      for (int a = 0; a < DIM; ++a) pj[a] = pn[a];
      const Tv xj = xn;
      if (v + 1 < nv) load(tc0, ntc, v + 1);
      else load(t0, nt, 0);
      const int col = tj + 8 * ((v & ~7) + ti);      // the column this lane writes
      const bool wr = dst && col < ntc;
      if ((v & 7) == 0 && !first) old = wr ? dst[col] : Tv(0);
      Tv cacc = Tv(0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        double r2 = 0.0;
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
          const double dx = pi[u][a] - pj[a];
          if (a == 0) r2 = MINED ? __builtin_fma(dx, dx, double(MIN_R2<Tv>)) : dx * dx;
          else r2 = __builtin_fma(dx, dx, r2);
        }
        const Tv k = kernel_fixed<KIND, DERIV, Tv, MINED, NORMAL>(kc, Tv(r2));
        racc[u] += k * xj;
        cacc += k * xi[u];
      }
      cacc = sum8(cacc);
      keep = ti == (v & 7) ? cacc : keep;
      if (((v & 7) == 7 || v + 1 == nv) && wr) {
        if (A.scale) keep *= Tv(A.scale[tc0 + col]);
        dst[col] = first ? keep : old + keep;
      }
    }
  }
  // row sums over the lanes of a row; lane (ti, tj) ends with row ti + 8 tj
  const Tv s = transpose_reduce_a<8, Tv>(racc, tj);
  const int i = ti + 8 * tj;
  if (i < nrow) {
    const int64_t gi = s0 + i;
    Tv o = A.scale ? Tv(A.scale[gi]) * s : s;
    if (A.pair_slot[p0] < 0) o += Tv(A.kp.shift) * A.x[gi];   // the diagonal pair comes first
    A.partial[int64_t(task) * A.ld + rt + i] = o;
  }
}

// Wave w: task w / nsplit, row chunks w % nsplit, + nsplit, ... of `chunk`
// rows each (chunk <= 64, a multiple of 8).  With nsplit = 1 one wave does a
// leaf's chunks in turn and adds their column sums; else each chunk has its
// own place, and a chunk beyond a shorter leaf's rows writes zeros.
template <typename Tv, int KIND, int DERIV, bool NORMAL>
__device__ __forceinline__ void near_wave(int wave, const int* __restrict__ tasks, int ntasks, const NearIn<Tv>& A,
                                          int dim, int chunk, int nchunk, bool mined) {
  constexpr bool MAY = KIND != KER_LAPLACE && DERIV != DER_RADIAL;   // no question about r = 0
  if (wave >= ntasks * A.nsplit) return;
  const int task = wave / A.nsplit, part = wave % A.nsplit;
  const int sl = tasks[3 * task], p0 = tasks[3 * task + 1], p1 = tasks[3 * task + 2];
  const int ns = A.leaf_off[sl + 1] - A.leaf_off[sl];
  for (int c = part; c < nchunk; c += A.nsplit) {
    const int rt = c * chunk, nrow = min(chunk, ns - rt);
    if (nrow <= 0) {
      if (A.nsplit > 1)
        for (int p = p0; p < p1; ++p)
          if (A.pair_slot[p] >= 0)
            for (int j = threadIdx.x & 63; j < A.ld; j += 64)
              A.colpart[(int64_t(A.pair_slot[p]) * A.nsplit + part) * A.ld + j] = Tv(0);
      continue;
    }
    auto run = [&](auto uc) {
      constexpr int U = decltype(uc)::value;
      if (dim == 3) near_rows<U, 3, MAY, NORMAL, Tv, KIND, DERIV>(A, task, part, sl, p0, p1, rt, nrow, c == part);
      else near_rows<U, 2, MAY, NORMAL, Tv, KIND, DERIV>(A, task, part, sl, p0, p1, rt, nrow, c == part);
    };
    // points on a line, and distances beyond any use: one loop for every length
    if (dim == 1) {
      near_rows<8, 1, false, NORMAL, Tv, KIND, DERIV>(A, task, part, sl, p0, p1, rt, nrow, c == part);
      continue;
    }
    if (MAY && !mined) {
      if (dim == 3) near_rows<8, 3, false, NORMAL, Tv, KIND, DERIV>(A, task, part, sl, p0, p1, rt, nrow, c == part);
      else near_rows<8, 2, false, NORMAL, Tv, KIND, DERIV>(A, task, part, sl, p0, p1, rt, nrow, c == part);
      continue;
    }
    switch ((nrow + 7) >> 3) {
      case 1: run(std::integral_constant<int, 1>{}); break;
      case 2: run(std::integral_constant<int, 2>{}); break;
      case 3: run(std::integral_constant<int, 3>{}); break;
      case 4: run(std::integral_constant<int, 4>{}); break;
      case 5: run(std::integral_constant<int, 5>{}); break;
      case 6: run(std::integral_constant<int, 6>{}); break;
      case 7: run(std::integral_constant<int, 7>{}); break;
      default: run(std::integral_constant<int, 8>{}); break;
    }
  }
}

template <typename Tv, int KIND, int DERIV, bool NORMAL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void
k_near(const int* __restrict__ tasks, int ntasks, NearIn<Tv> A, int dim, int chunk, int nchunk, bool mined) {
  near_wave<Tv, KIND, DERIV, NORMAL>(wave_id(), tasks, ntasks, A, dim, chunk, nchunk, mined);
}

// Near field and couplings of a fine FP64 product in one launch.  The first is
// bound by vector issue, the second by HBM, and neither needs the other.
// far_share: 2^32 times the share of the coupling blocks, rounded up, which
// spreads them evenly over the launch.  (On two streams nothing overlapped: the
// near field of the one took every wave slot before the other started.)
// Registers for three waves a SIMD, as the near field alone, so a 64 x 64 tile
// is read in two halves; the coupling waves go first when their data is there.
// A product of 131072 points (3D, rank 64) took 2438 us with two launches and
// 2246 with one (2136 since the entries take one operation less), 50000 points (rank 27 in tiles of 32) 593 and 566; with
// tiles of 16, which want more waves in flight than three, 90000 points took 190
// and 199 us, 4096 points 35.6 and 36.8: those stay two launches.
struct FarIn {
  const int* tasks;
  int ntasks;
  const double* blk;
  const int* blk_col;
  const int* blk_slot;
  const double* x;
  double* partial;
  double* colpart;
  int r, T;
};

template <int KIND>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void
k_near_far(const int* __restrict__ tasks, int ntasks, NearIn<double> A, int dim, int chunk, int nchunk, bool mined,
           FarIn F, uint32_t far_share) {
  const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  const uint32_t b = blockIdx.x, f = __umulhi(b, far_share);
  if (__umulhi(b + 1, far_share) == f) {
    near_wave<double, KIND, DER_NONE, true>(int(b - f) * 4 + wv, tasks, ntasks, A, dim, chunk, nchunk, mined);
    return;
  }
  __builtin_amdgcn_s_setprio(3);         // few instructions, each behind a load
  auto go = [&](auto tc, auto fullc) {
    constexpr int T = decltype(tc)::value;
    constexpr bool FULL = decltype(fullc)::value;
    bsr_gemv_wave<T, FULL, T == 8 ? 2 : 1, double, double>(int(f) * 4 + wv, F.tasks, F.ntasks, F.blk, F.blk_col,
                                                           F.blk_slot, F.x, F.partial, F.colpart, F.r,
                                                           FULL ? 8 : tile_A(F.r, T));
  };
  auto pick = [&](auto tc) {
    if (F.r == 8 * decltype(tc)::value) go(tc, std::true_type{});
    else go(tc, std::false_type{});
  };
  if (F.T == 4) pick(std::integral_constant<int, 4>{});
  else pick(std::integral_constant<int, 8>{});
}

}  // namespace

bool launch_near_far(H2& h, const void* xtree, const Launch& l, const void* xall) {
  const NearField& nf = h.near;
  if (h.T < 4 || h.nq > 0 || h.timing || h.kp.deriv != DER_NONE || nf.ntasks == 0 || l.ntasks == 0) return false;
  const int64_t nn = (int64_t(nf.ntasks) * nf.nsplit + 3) / 4, nfar = (l.ntasks + 3) / 4;
  const uint32_t share = uint32_t((uint64_t(nfar) << 32) / uint64_t(nn + nfar) + 1);
  KernelParams kp = h.kp;
  if (h.diag) kp.shift = 0.0;          // the per-point diagonal is added by k_fine_reduce
  const NearIn<double> A{nf.pair_col, nf.pair_slot, h.leaf_off, h.pts, h.scale, static_cast<const double*>(xtree),
                         h.near_partial, h.near_colpart, kp, nf.ld, nf.nsplit};
  const FarIn F{l.task, l.ntasks, static_cast<const double*>(h.prec[P64].blk), h.blk_col, h.blk_slot,
                static_cast<const double*>(xall), h.partial, h.colpart, h.r, h.T};
  auto go = [&](auto kc) {
    hipLaunchKernelGGL((k_near_far<decltype(kc)::value>), dim3(unsigned(nn + nfar)), dim3(256), 0, h.stream, nf.task,
                       nf.ntasks, A, h.dim, nf.chunk, nf.nchunk, nf.mined, F, share);
  };
  switch (h.kp.kind) {
    case KER_EXP: go(std::integral_constant<int, KER_EXP>{}); break;
    case KER_GAUSS: go(std::integral_constant<int, KER_GAUSS>{}); break;
    case KER_LAPLACE: go(std::integral_constant<int, KER_LAPLACE>{}); break;
    default: go(std::integral_constant<int, KER_MATERN32>{}); break;
  }
  check_launch("near_far");
  return true;
}

void launch_near(H2& h, int p, const void* xtree) {
  if (h.nq > 0) throw std::runtime_error("close entries by quadrature are applied from the stored tiles only");
  const NearField& nf = h.near;
  if (nf.ntasks == 0) return;
  int ev;
  h.time_begin(ev);
  const dim3 g(unsigned((int64_t(nf.ntasks) * nf.nsplit + 3) / 4)), b(256);
  KernelParams kp = h.kp;
  if (h.diag) kp.shift = 0.0;          // the per-point diagonal is added by k_fine_reduce
  auto go = [&](auto tv, auto kc, auto dc, auto nc) {
    using Tv = decltype(tv);
    constexpr int K = decltype(kc)::value, D = decltype(dc)::value;
    const NearIn<Tv> A{nf.pair_col, nf.pair_slot, h.leaf_off, h.pts, h.scale, static_cast<const Tv*>(xtree),
                       reinterpret_cast<Tv*>(h.near_partial), reinterpret_cast<Tv*>(h.near_colpart), kp, nf.ld,
                       nf.nsplit};
    hipLaunchKernelGGL((k_near<Tv, K, D, decltype(nc)::value>), g, b, 0, h.stream, nf.task, nf.ntasks, A, h.dim,
                       nf.chunk, nf.nchunk, nf.mined);
  };
  dispatch_kernel(h.kp.kind, h.kp.deriv, [&](auto kc, auto dc) {
    if (p == P64) go(double{}, kc, dc, std::true_type{});
    else if (nf.normal32) go(float{}, kc, dc, std::true_type{});
    else go(float{}, kc, dc, std::false_type{});
  });
  check_launch("near");
  h.time_end(p == P64 ? KS_NEAR64 : KS_NEAR32, ev, double(h.near_evals));
}

}  // namespace h2mg
