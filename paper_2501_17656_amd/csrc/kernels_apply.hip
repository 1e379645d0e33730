// Apply kernels of the H2 matvec and of the restricted operators.
//
// Section 3.1: y = A x is computed by the upsweep x_i = V_i x_{i-1} (leaf
// bases then transfers), the per-level coupling products, the downsweep
// y_{i-1} = D_i x_{i-1} + U_i y_i, and the close (near-field) leaf blocks
// y = D x + U_1 y_1.  Section 3.3: a restricted operator A_k has the same
// structure with the projected close blocks of its depth in place of D.
//
// Every r x r block product is HBM-bound (one FMA per stored word), so the
// blocks are stored once (upper triangle, symmetric operators) in the tiled
// layout of device_common.h and each wave streams one run of blocks of a
// block row: it accumulates B x_t for the row in registers and emits
// B^T x_s for the block's column, which a reduce pass gathers in a fixed
// order (deterministic, no atomics).
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

// Couplings and projected close blocks (r x r tiles).
template <int T, bool FULL, typename Tb, typename Tv>
__global__ __launch_bounds__(256) void k_bsr_gemv(const int* __restrict__ tasks, int ntasks,
                                                  const Tb* __restrict__ blk,
                                                  const int* __restrict__ blk_col,
                                                  const int* __restrict__ blk_slot,
                                                  const Tv* __restrict__ x, Tv* __restrict__ partial,
                                                  Tv* __restrict__ colpart, int r) {
  bsr_gemv_wave<T, FULL, 1, Tb, Tv>(wave_id(), tasks, ntasks, blk, blk_col, blk_slot, x, partial, colpart, r,
                                 FULL ? 8 : tile_A(r, T));
}

// Stored near field: 64 x 64 FP64 tiles between leaf chunks (same body; a
// kernel of its own so profiles separate it from the coupling products).
__global__ __launch_bounds__(256) void k_near_gemv(const int* __restrict__ tasks, int ntasks,
                                                   const double* __restrict__ tiles,
                                                   const int* __restrict__ blk_col,
                                                   const int* __restrict__ blk_slot,
                                                   const double* __restrict__ x,
                                                   double* __restrict__ partial,
                                                   double* __restrict__ colpart, int A) {
  bsr_gemv_wave<8, true, 1, double, double>(wave_id(), tasks, ntasks, tiles, blk_col, blk_slot, x, partial,
                                         colpart, 64, A);
}

// The same over FP32 copies of the tiles (close entries given by quadrature,
// which the FP32 products cannot evaluate on the fly).
__global__ __launch_bounds__(256) void k_near_gemv32(const int* __restrict__ tasks, int ntasks,
                                                     const float* __restrict__ tiles,
                                                     const int* __restrict__ blk_col,
                                                     const int* __restrict__ blk_slot,
                                                     const float* __restrict__ x,
                                                     float* __restrict__ partial,
                                                     float* __restrict__ colpart, int A) {
  bsr_gemv_wave<8, true, 1, float, float>(wave_id(), tasks, ntasks, tiles, blk_col, blk_slot, x, partial, colpart, 64, A);
}

// Sources of one depth for the reduce: task partials of the row (contiguous
// in the launch) and column contributions (contiguous slots).
struct RedDepth {
  const int* rtp[2];     // row -> task offsets within the view
  const int* cptr[2];    // row -> column-slot offsets within the view
  int base[2];           // task base of the view in the GEMV launch
  int slot[2];           // slot base of the view
  int nsrc;
  int row0;              // first grid row of this depth
  int64_t out_off;       // element offset of the depth in the output buffer
};
constexpr int MAX_RED_DEPTHS = 20;
struct RedArgs {
  RedDepth dep[MAX_RED_DEPTHS];
  int ndep;
  int nrows;
};

// v += p[t * stride] for t in [a, b), four loads in flight, in a fixed order.
template <typename Tv>
__device__ __forceinline__ void sum_run(Tv& v, const Tv* __restrict__ p, int64_t stride, int64_t a, int64_t b) {
  Tv v0 = zero<Tv>(), v1 = zero<Tv>(), v2 = zero<Tv>(), v3 = zero<Tv>();
  int64_t t = a;
  for (; t + 4 <= b; t += 4) {
    v0 += p[t * stride];
    v1 += p[(t + 1) * stride];
    v2 += p[(t + 2) * stride];
    v3 += p[(t + 3) * stride];
  }
  for (; t < b; ++t) v0 += p[t * stride];
  v += (v0 + v1) + (v2 + v3);
}

// One workgroup per row of any depth: out = sum of its partials, in a fixed
// order.  A row has up to some hundred contributions and moves little, so the
// length of the chain of loads is what counts: the 256 threads are 256 / rp
// groups (rp: the power of two that holds r), each sums its share of every
// list with four loads in flight, and the groups' sums meet in LDS.  With one
// wave per row the reduces were a tenth of a solve on 65536 points (23 us
// each; 10 us now).
template <typename Tv>
__global__ __launch_bounds__(256) void k_reduce(RedArgs A, const Tv* __restrict__ partial,
                                                const Tv* __restrict__ colpart, Tv* __restrict__ out,
                                                Tv* __restrict__ out_last, int r, int rp) {
  __shared__ Tv red[256];
  const int grow = blockIdx.x;
  int q = 0;
  while (q + 1 < A.ndep && A.dep[q + 1].row0 <= grow) ++q;
  const RedDepth& D = A.dep[q];
  const int row = grow - D.row0;
  const int i = threadIdx.x & (rp - 1), g = threadIdx.x / rp, ng = 256 / rp;
  Tv v = zero<Tv>();
  if (i < r) {
    for (int sidx = 0; sidx < D.nsrc; ++sidx) {
      const int64_t t0 = D.rtp[sidx][row], nt = D.rtp[sidx][row + 1] - t0;
      sum_run(v, partial + int64_t(D.base[sidx]) * r + i, r, t0 + g * nt / ng, t0 + (g + 1) * nt / ng);
      const int64_t c0 = D.cptr[sidx][row], nc = D.cptr[sidx][row + 1] - c0;
      sum_run(v, colpart + int64_t(D.slot[sidx]) * r + i, r, c0 + g * nc / ng, c0 + (g + 1) * nc / ng);
    }
  }
  red[threadIdx.x] = v;
  __syncthreads();
  if (threadIdx.x >= r) return;
  for (int k = 1; k < ng; ++k) v += red[k * rp + threadIdx.x];
  if (out_last && q == A.ndep - 1) out_last[int64_t(row) * r + i] = v;
  else out[D.out_off + int64_t(row) * r + i] = v;
}

// ------------------------------------------------------------ transfers
// xpar[s] = sum_c E_c^T xchild[c] over the two children of s (depth d -> d+1 kids).
template <int T, typename Tb, typename Tv>
__global__ __launch_bounds__(256) void k_transfer_up(int nparents, int gidc0,
                                                     const Tb* __restrict__ E,
                                                     const Tv* __restrict__ xchild,
                                                     Tv* __restrict__ xpar, int r) {
  const int s = int((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  if (s >= nparents) return;
  const int lane = threadIdx.x & 63;
  const int a = lane >> 3, b = lane & 7;
  Tv z[T];
#pragma unroll
  for (int v = 0; v < T; ++v) z[v] = zero<Tv>();
  for (int q = 0; q < 2; ++q) {
    const int c = 2 * s + q;
    Tv xs[T];
#pragma unroll
    for (int u = 0; u < T; ++u) {
      const int i = a * T + u;
      xs[u] = i < r ? xchild[int64_t(c) * r + i] : zero<Tv>();
    }
    Tv B[T * T];
    load_subtile<T, Tb, Tv>(E + int64_t(gidc0 + c) * tile_elems(T), lane, tile_A(r, T), B);
#pragma unroll
    for (int v = 0; v < T; ++v)
#pragma unroll
      for (int u = 0; u < T; ++u) z[v] += B[u * T + v] * xs[u];
  }
#pragma unroll
  for (int v = 0; v < T; ++v) {
    Tv s2 = z[v];
    s2 += shfl_xor(s2, 8);
    s2 += shfl_xor(s2, 16);
    s2 += shfl_xor(s2, 32);
    z[v] = s2;
  }
  if (a == 0) {
#pragma unroll
    for (int v = 0; v < T; ++v) {
      const int j = b * T + v;
      if (j < r) xpar[int64_t(s) * r + j] = z[v];
    }
  }
}

// ychild[c] = addend[c] + E_c ypar[c / 2] for every child c at depth d+1.
template <int T, typename Tb, typename Tv>
__global__ __launch_bounds__(256) void k_transfer_down(int nchildren, int gidc0,
                                                       const Tb* __restrict__ E,
                                                       const Tv* __restrict__ ypar,
                                                       Tv* __restrict__ ychild,
                                                       const Tv* __restrict__ addend, int r) {
  const int c = int((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  if (c >= nchildren) return;
  const int lane = threadIdx.x & 63;
  const int a = lane >> 3, b = lane & 7;
  const int s = c >> 1;
  Tv xt[T];
#pragma unroll
  for (int v = 0; v < T; ++v) {
    const int j = b * T + v;
    xt[v] = j < r ? ypar[int64_t(s) * r + j] : zero<Tv>();
  }
  Tv B[T * T];
  load_subtile<T, Tb, Tv>(E + int64_t(gidc0 + c) * tile_elems(T), lane, tile_A(r, T), B);
  Tv acc[T];
#pragma unroll
  for (int u = 0; u < T; ++u) {
    Tv s2 = zero<Tv>();
#pragma unroll
    for (int v = 0; v < T; ++v) s2 += B[u * T + v] * xt[v];
    s2 += shfl_xor(s2, 1);
    s2 += shfl_xor(s2, 2);
    s2 += shfl_xor(s2, 4);
    acc[u] = s2;
  }
  if (b == 0) {
#pragma unroll
    for (int u = 0; u < T; ++u) {
      const int i = a * T + u;
      if (i < r)
        ychild[int64_t(c) * r + i] = acc[u] + (addend ? addend[int64_t(c) * r + i] : zero<Tv>());
    }
  }
}

// ------------------------------------------------------------ leaf bases
// xhat[leaf] = Q_leaf^T x_leaf; 256 / rp groups (rp: the power of two that
// holds r) split the leaf's rows.  With perm, x is in user order and is
// written to xtree in tree order as well.
template <typename Tq, typename Tv>
__global__ __launch_bounds__(256) void k_leaf_up(const int* __restrict__ leaf_off,
                                                 const Tq* __restrict__ Qr,
                                                 const Tv* __restrict__ x, Tv* __restrict__ xhat,
                                                 int r, int rp, const int64_t* __restrict__ perm,
                                                 Tv* __restrict__ xtree) {
  __shared__ Tv red[256];
  __shared__ Tv xl[256];
  const int leaf = blockIdx.x, tid = threadIdx.x;
  const int s0 = leaf_off[leaf], n = leaf_off[leaf + 1] - s0;
  if (tid < n) {                       // at most 256 points
    const Tv v = perm ? x[perm[s0 + tid]] : x[s0 + tid];
    xl[tid] = v;
    if (perm) xtree[s0 + tid] = v;
  }
  __syncthreads();
  const int j = tid & (rp - 1), g = tid / rp, ng = 256 / rp;
  Tv acc = zero<Tv>();
  if (j < r) {
    const Tq* Q = Qr + int64_t(s0) * r + j;
#pragma unroll 4
    for (int i = g; i < n; i += ng) acc += ld_as<Tv, Tq>(Q[int64_t(i) * r]) * xl[i];
  }
  red[tid] = acc;
  __syncthreads();
  if (tid >= r) return;
  for (int k = 1; k < ng; ++k) acc += red[k * rp + tid];
  xhat[int64_t(leaf) * r + tid] = acc;
}

// ------------------------------------------------------------ fine output
// out[idx(i)] = alpha * (Q_leaf yhat_leaf + near sums)_i + beta * add[idx(i)]
// for 64 rows i of one leaf per workgroup; idx = i or perm[i].  The near sums
// are the row partials of the leaf's tasks and its column sums (nsplit per
// pair, ordered by column leaf), up to some hundred runs of one leaf's
// length.  Bound by latency, not bytes: the four waves take a quarter of the
// basis columns and of both lists each, with four loads in flight.  One
// thread per row summing all of them, each through an index, took 274 us on
// 50000 points of a Gaussian mixture; 28 us now.
template <typename Tq, typename Tv>
__global__ __launch_bounds__(256) void k_fine_reduce(
    const int* __restrict__ leaf_off, const Tq* __restrict__ Qc, const Tv* __restrict__ yhat, int r,
    const int* __restrict__ row_task_ptr, const int* __restrict__ col_ptr, int nsplit,
    const Tv* __restrict__ partial, const Tv* __restrict__ colpart, int ld, const Tv* __restrict__ near_y,
    const int* __restrict__ chunk_base, const double* __restrict__ dg, const Tv* __restrict__ xin,
    const int64_t* __restrict__ perm, Tv* __restrict__ out, double alpha, const Tv* __restrict__ add,
    double beta) {
  __shared__ Tv red[4][64];
  const int leaf = blockIdx.x;
  const int s0 = leaf_off[leaf], n = leaf_off[leaf + 1] - s0;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = 64 * int(blockIdx.y) + lane;
  if (64 * int(blockIdx.y) >= n) return;
  Tv v = zero<Tv>();
  if (i < n) {
    const Tq* Q = Qc + int64_t(s0) * r + i;
    const Tv* yh = yhat + int64_t(leaf) * r;
#pragma unroll 4
    for (int j = w * r / 4; j < (w + 1) * r / 4; ++j) v += ld_as<Tv, Tq>(Q[int64_t(j) * n]) * yh[j];
    if (near_y) {
      if (w == 0) v += near_y[chunk_pos(chunk_base[leaf], chunk_len(n), i)];
    } else {
      const int64_t t0 = row_task_ptr[leaf], nt = row_task_ptr[leaf + 1] - t0;
      const int64_t c0 = int64_t(col_ptr[leaf]) * nsplit, nc = int64_t(col_ptr[leaf + 1]) * nsplit - c0;
      sum_run(v, partial + i, ld, t0 + w * nt / 4, t0 + (w + 1) * nt / 4);
      sum_run(v, colpart + i, ld, c0 + w * nc / 4, c0 + (w + 1) * nc / 4);
      if (dg && w == 0) v += Tv(dg[s0 + i]) * xin[s0 + i];
    }
  }
  red[w][lane] = v;
  __syncthreads();
  if (w == 0 && i < n) {
    v = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
    const int64_t idx = perm ? perm[s0 + i] : int64_t(s0 + i);
    Tv o = Tv(alpha) * v;
    if (add) o += Tv(beta) * add[idx];
    out[idx] = o;
  }
}

// out[idx(i)] = alpha * (Q_leaf yhat_leaf)_i + beta * add[idx(i)] (prolongation
// from the depth-L coefficients to the points; tree order).
template <typename Tq, typename Tv>
__global__ __launch_bounds__(256) void k_leaf_down(const int* __restrict__ leaf_off,
                                                   const Tq* __restrict__ Qc,
                                                   const Tv* __restrict__ yhat, int r,
                                                   Tv* __restrict__ out, double alpha,
                                                   const Tv* __restrict__ add, double beta) {
  __shared__ Tv yh[64];
  const int leaf = blockIdx.x;
  const int s0 = leaf_off[leaf], n = leaf_off[leaf + 1] - s0;
  if (threadIdx.x < r) yh[threadIdx.x] = yhat[int64_t(leaf) * r + threadIdx.x];
  __syncthreads();
  const Tq* Q = Qc + int64_t(s0) * r;
  for (int i = threadIdx.x; i < n; i += 256) {
    Tv v = zero<Tv>();
    for (int j = 0; j < r; ++j) v += ld_as<Tv, Tq>(Q[int64_t(j) * n + i]) * yh[j];
    Tv o = Tv(alpha) * v;
    if (add) o += Tv(beta) * add[s0 + i];
    out[s0 + i] = o;
  }
}

// The tree-order vector in the chunk-padded layout of the stored near field
// (padding entries are never written and stay zero).
template <typename Tv>
__global__ __launch_bounds__(256) void k_near_pad(const int* __restrict__ leaf_off,
                                                  const int* __restrict__ chunk_base,
                                                  const Tv* __restrict__ x,
                                                  Tv* __restrict__ xc) {
  const int leaf = blockIdx.x;
  const int s0 = leaf_off[leaf], n = leaf_off[leaf + 1] - s0;
  const int len = chunk_len(n);
  for (int i = threadIdx.x; i < n; i += 256) xc[chunk_pos(chunk_base[leaf], len, i)] = x[s0 + i];
}

// ------------------------------------------------------------ dispatch helpers
template <typename F>
void dispatch_T(int T, F&& f) {
  switch (T) {
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    default: f(std::integral_constant<int, 8>{}); break;
  }
}

inline int grid_waves(int64_t waves) { return int((waves + 3) / 4); }

}  // namespace

// ------------------------------------------------------------ launchers
void launch_gemv(H2& h, int p, const Launch& l, const void* x_all) {
  if (l.ntasks == 0) return;
  int ev;
  h.time_begin(ev);
  dispatch_T(h.T, [&](auto Tc) {
    constexpr int T = decltype(Tc)::value;
    const dim3 g(grid_waves(l.ntasks)), b(256);
    auto go = [&](auto fullc) {
      constexpr bool F = decltype(fullc)::value;
      if (p == P64)
        hipLaunchKernelGGL((k_bsr_gemv<T, F, double, double>), g, b, 0, h.stream, l.task, l.ntasks,
                           static_cast<const double*>(h.prec[P64].blk), h.blk_col, h.blk_slot,
                           static_cast<const double*>(x_all), h.partial, h.colpart, h.r);
      else if (p == P32)
        hipLaunchKernelGGL((k_bsr_gemv<T, F, float, float>), g, b, 0, h.stream, l.task, l.ntasks,
                           static_cast<const float*>(h.prec[P32].blk), h.blk_col, h.blk_slot,
                           static_cast<const float*>(x_all), reinterpret_cast<float*>(h.partial),
                           reinterpret_cast<float*>(h.colpart), h.r);
      else
        hipLaunchKernelGGL((k_bsr_gemv<T, F, bf16, float>), g, b, 0, h.stream, l.task, l.ntasks,
                           static_cast<const bf16*>(h.prec[P16].blk), h.blk_col, h.blk_slot,
                           static_cast<const float*>(x_all), reinterpret_cast<float*>(h.partial),
                           reinterpret_cast<float*>(h.colpart), h.r);
    };
    if (h.r == 8 * T) go(std::true_type{});
    else go(std::false_type{});
  });
  check_launch("bsr_gemv");
  h.time_end(KS_GEMV64 + p, ev, double(l.nblocks) * h.r * h.r * elem_bytes(p));
}

void launch_reduce(H2& h, int p, int d0, int d1, const View* const* v0, const int* base0,
                   const View* const* v1, const int* base1, void* out, void* out_last) {
  RedArgs A{};
  A.ndep = d1 - d0 + 1;
  if (A.ndep > MAX_RED_DEPTHS) throw std::runtime_error("too many depths for one reduce");
  int rows = 0;
  for (int q = 0; q < A.ndep; ++q) {
    const int d = d0 + q;
    RedDepth& D = A.dep[q];
    D.rtp[0] = v0[q]->row_task_ptr;
    D.cptr[0] = v0[q]->col_ptr;
    D.base[0] = base0[q];
    D.slot[0] = v0[q]->slot_base;
    D.nsrc = 1;
    if (v1 && v1[q]) {
      D.rtp[1] = v1[q]->row_task_ptr;
      D.cptr[1] = v1[q]->col_ptr;
      D.base[1] = base1[q];
      D.slot[1] = v1[q]->slot_base;
      D.nsrc = 2;
    }
    D.row0 = rows;
    D.out_off = int64_t((1 << d) - 1) * h.r;
    rows += 1 << d;
  }
  A.nrows = rows;
  const dim3 g(rows), b(256);
  if (p == P64)
    hipLaunchKernelGGL(k_reduce<double>, g, b, 0, h.stream, A, h.partial, h.colpart,
                       static_cast<double*>(out), static_cast<double*>(out_last), h.r, 8 * h.T);
  else
    hipLaunchKernelGGL(k_reduce<float>, g, b, 0, h.stream, A, reinterpret_cast<const float*>(h.partial),
                       reinterpret_cast<const float*>(h.colpart), static_cast<float*>(out),
                       static_cast<float*>(out_last), h.r, 8 * h.T);
  check_launch("reduce");
}

void launch_transfer_up(H2& h, int p, int d, const void* xchild, void* xpar) {
  const int npar = 1 << d;
  const int gidc0 = (1 << (d + 1)) - 1;
  dispatch_T(h.T, [&](auto Tc) {
    constexpr int T = decltype(Tc)::value;
    const dim3 g(grid_waves(npar)), b(256);
    if (p == P64)
      hipLaunchKernelGGL((k_transfer_up<T, double, double>), g, b, 0, h.stream, npar, gidc0,
                         static_cast<const double*>(h.prec[P64].E), static_cast<const double*>(xchild),
                         static_cast<double*>(xpar), h.r);
    else if (p == P32)
      hipLaunchKernelGGL((k_transfer_up<T, float, float>), g, b, 0, h.stream, npar, gidc0,
                         static_cast<const float*>(h.prec[P32].E), static_cast<const float*>(xchild),
                         static_cast<float*>(xpar), h.r);
    else
      hipLaunchKernelGGL((k_transfer_up<T, bf16, float>), g, b, 0, h.stream, npar, gidc0,
                         static_cast<const bf16*>(h.prec[P16].E), static_cast<const float*>(xchild),
                         static_cast<float*>(xpar), h.r);
  });
  check_launch("transfer_up");
}

void launch_transfer_down(H2& h, int p, int d, const void* ypar, void* ychild, const void* addend) {
  const int nch = 1 << (d + 1);
  const int gidc0 = (1 << (d + 1)) - 1;
  dispatch_T(h.T, [&](auto Tc) {
    constexpr int T = decltype(Tc)::value;
    const dim3 g(grid_waves(nch)), b(256);
    if (p == P64)
      hipLaunchKernelGGL((k_transfer_down<T, double, double>), g, b, 0, h.stream, nch, gidc0,
                         static_cast<const double*>(h.prec[P64].E), static_cast<const double*>(ypar),
                         static_cast<double*>(ychild), static_cast<const double*>(addend), h.r);
    else if (p == P32)
      hipLaunchKernelGGL((k_transfer_down<T, float, float>), g, b, 0, h.stream, nch, gidc0,
                         static_cast<const float*>(h.prec[P32].E), static_cast<const float*>(ypar),
                         static_cast<float*>(ychild), static_cast<const float*>(addend), h.r);
    else
      hipLaunchKernelGGL((k_transfer_down<T, bf16, float>), g, b, 0, h.stream, nch, gidc0,
                         static_cast<const bf16*>(h.prec[P16].E), static_cast<const float*>(ypar),
                         static_cast<float*>(ychild), static_cast<const float*>(addend), h.r);
  });
  check_launch("transfer_down");
}

void launch_leaf_up(H2& h, int p, const void* xtree, void* xhat) {
  const dim3 g(h.nleaf), b(256);
  if (p == P64)
    hipLaunchKernelGGL((k_leaf_up<double, double>), g, b, 0, h.stream, h.leaf_off,
                       static_cast<const double*>(h.prec[P64].Qr), static_cast<const double*>(xtree),
                       static_cast<double*>(xhat), h.r, 8 * h.T, static_cast<const int64_t*>(nullptr),
                       static_cast<double*>(nullptr));
  else if (p == P32)
    hipLaunchKernelGGL((k_leaf_up<float, float>), g, b, 0, h.stream, h.leaf_off,
                       static_cast<const float*>(h.prec[P32].Qr), static_cast<const float*>(xtree),
                       static_cast<float*>(xhat), h.r, 8 * h.T, static_cast<const int64_t*>(nullptr),
                       static_cast<float*>(nullptr));
  else
    hipLaunchKernelGGL((k_leaf_up<bf16, float>), g, b, 0, h.stream, h.leaf_off,
                       static_cast<const bf16*>(h.prec[P16].Qr), static_cast<const float*>(xtree),
                       static_cast<float*>(xhat), h.r, 8 * h.T, static_cast<const int64_t*>(nullptr),
                       static_cast<float*>(nullptr));
  check_launch("leaf_up");
}

void launch_leaf_up_gather(H2& h, const double* xuser, double* xtree, double* xhat) {
  hipLaunchKernelGGL((k_leaf_up<double, double>), dim3(h.nleaf), dim3(256), 0, h.stream, h.leaf_off,
                     static_cast<const double*>(h.prec[P64].Qr), xuser, xhat, h.r, 8 * h.T,
                     static_cast<const int64_t*>(h.perm), xtree);
  check_launch("leaf_up_gather");
}

void launch_near_stored(H2& h, int p, const void* xtree) {
  StoredNear& sn = h.snear;
  if (sn.nblocks == 0) return;
  if (p != P64 && !sn.tiles32) throw std::runtime_error("no FP32 copy of the stored near field");
  RedArgs A{};
  A.ndep = 1;
  A.nrows = sn.nchunk;
  RedDepth& D = A.dep[0];
  D.rtp[0] = sn.row_task_ptr;
  D.cptr[0] = sn.col_ptr;
  D.base[0] = 0;
  D.slot[0] = 0;
  D.nsrc = 1;
  D.row0 = 0;
  D.out_off = 0;
  if (p == P64) {
    const double* xc = static_cast<const double*>(xtree);
    if (!sn.identity) {
      hipLaunchKernelGGL(k_near_pad<double>, dim3(h.nleaf), dim3(256), 0, h.stream, h.leaf_off,
                         sn.chunk_base, xc, sn.xc);
      check_launch("near_pad");
      xc = sn.xc;
    }
    int ev;
    h.time_begin(ev);
    hipLaunchKernelGGL(k_near_gemv, dim3(grid_waves(sn.ntasks)), dim3(256), 0, h.stream, sn.task,
                       sn.ntasks, sn.tiles, sn.blk_col, sn.blk_slot, xc, sn.partial, sn.colpart, sn.lanes);
    check_launch("near_gemv");
    h.time_end(KS_NEARST64, ev, double(sn.nblocks) * (64.0 * sn.lanes * sn.lanes) * sizeof(double));
    hipLaunchKernelGGL(k_reduce<double>, dim3(sn.nchunk), dim3(256), 0, h.stream, A,
                       sn.partial, sn.colpart, sn.yc, static_cast<double*>(nullptr), 64, 64);
  } else {
    // FP32 partials and output in the first half of the FP64 buffers; the
    // padded input has a zero-padded FP32 buffer of its own
    const float* xc = static_cast<const float*>(xtree);
    if (!sn.identity) {
      hipLaunchKernelGGL(k_near_pad<float>, dim3(h.nleaf), dim3(256), 0, h.stream, h.leaf_off,
                         sn.chunk_base, xc, sn.xc32);
      check_launch("near_pad");
      xc = sn.xc32;
    }
    float* part = reinterpret_cast<float*>(sn.partial);
    float* cpart = reinterpret_cast<float*>(sn.colpart);
    hipLaunchKernelGGL(k_near_gemv32, dim3(grid_waves(sn.ntasks)), dim3(256), 0, h.stream, sn.task,
                       sn.ntasks, sn.tiles32, sn.blk_col, sn.blk_slot, xc, part, cpart, sn.lanes);
    check_launch("near_gemv32");
    hipLaunchKernelGGL(k_reduce<float>, dim3(sn.nchunk), dim3(256), 0, h.stream, A,
                       static_cast<const float*>(part), static_cast<const float*>(cpart),
                       reinterpret_cast<float*>(sn.yc), static_cast<float*>(nullptr), 64, 64);
  }
  check_launch("near_reduce");
}

void launch_fine_reduce(H2& h, int p, const void* yhat, void* out, bool to_user, double alpha,
                        const void* add, double beta, const void* xin) {
  const dim3 g(h.nleaf, (h.leaf_max + 63) / 64), b(256);
  const int64_t* perm = to_user ? h.perm : nullptr;
  const bool stored = near_stored_for(h, p);
  const double* dg = stored ? nullptr : h.diag;     // stored tiles hold the diagonal
  if (p == P64)
    hipLaunchKernelGGL((k_fine_reduce<double, double>), g, b, 0, h.stream, h.leaf_off,
                       static_cast<const double*>(h.prec[P64].Qc), static_cast<const double*>(yhat),
                       h.r, h.near.row_task_ptr, h.near.col_ptr, h.near.nsplit, h.near_partial,
                       h.near_colpart, h.near.ld, stored ? h.snear.yc : nullptr, h.snear.chunk_base, dg,
                       static_cast<const double*>(xin), perm, static_cast<double*>(out), alpha,
                       static_cast<const double*>(add), beta);
  else if (p == P32)
    hipLaunchKernelGGL((k_fine_reduce<float, float>), g, b, 0, h.stream, h.leaf_off,
                       static_cast<const float*>(h.prec[P32].Qc), static_cast<const float*>(yhat),
                       h.r, h.near.row_task_ptr, h.near.col_ptr, h.near.nsplit,
                       reinterpret_cast<const float*>(h.near_partial),
                       reinterpret_cast<const float*>(h.near_colpart), h.near.ld,
                       stored ? reinterpret_cast<const float*>(h.snear.yc) : nullptr, h.snear.chunk_base, dg,
                       static_cast<const float*>(xin), perm, static_cast<float*>(out), alpha,
                       static_cast<const float*>(add), beta);
  else
    hipLaunchKernelGGL((k_fine_reduce<bf16, float>), g, b, 0, h.stream, h.leaf_off,
                       static_cast<const bf16*>(h.prec[P16].Qc), static_cast<const float*>(yhat),
                       h.r, h.near.row_task_ptr, h.near.col_ptr, h.near.nsplit,
                       reinterpret_cast<const float*>(h.near_partial),
                       reinterpret_cast<const float*>(h.near_colpart), h.near.ld,
                       stored ? reinterpret_cast<const float*>(h.snear.yc) : nullptr, h.snear.chunk_base, dg,
                       static_cast<const float*>(xin), perm, static_cast<float*>(out), alpha,
                       static_cast<const float*>(add), beta);
  check_launch("fine_reduce");
}

void launch_leaf_down(H2& h, int p, const void* yhat, void* out, double alpha, const void* add,
                      double beta) {
  const dim3 g(h.nleaf), b(256);
  if (p == P64)
    hipLaunchKernelGGL((k_leaf_down<double, double>), g, b, 0, h.stream, h.leaf_off,
                       static_cast<const double*>(h.prec[P64].Qc), static_cast<const double*>(yhat),
                       h.r, static_cast<double*>(out), alpha, static_cast<const double*>(add), beta);
  else if (p == P32)
    hipLaunchKernelGGL((k_leaf_down<float, float>), g, b, 0, h.stream, h.leaf_off,
                       static_cast<const float*>(h.prec[P32].Qc), static_cast<const float*>(yhat),
                       h.r, static_cast<float*>(out), alpha, static_cast<const float*>(add), beta);
  else
    hipLaunchKernelGGL((k_leaf_down<bf16, float>), g, b, 0, h.stream, h.leaf_off,
                       static_cast<const bf16*>(h.prec[P16].Qc), static_cast<const float*>(yhat),
                       h.r, static_cast<float*>(out), alpha, static_cast<const float*>(add), beta);
  check_launch("leaf_down");
}

}  // namespace h2mg
