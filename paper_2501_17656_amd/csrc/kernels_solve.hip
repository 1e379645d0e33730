// Vector kernels of the V-cycle: permutations, axpby, FP64-accumulated dot
// products, the two halves of a CG step with device-resident scalars, and
// the triangular solves with the Cholesky factor of the coarsest operator.
//
// Section 3.3: the smoother Iter(A, r, e0) is CG, and the coarsest level is
// solved directly with a Cholesky factorisation.  Dot products are reduced
// in two fixed-order stages (per-workgroup partials, then a one-wave sum in
// the consumer) so results are deterministic and no host round trip is
// needed between CG steps.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <stdexcept>
#include <string>

#include "h2_impl.h"

namespace h2mg {

namespace {

constexpr int NT = 256;
constexpr int MAX_PARTS = DOT_PARTS;

void check_launch(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) throw std::runtime_error(std::string(what) + ": " + hipGetErrorString(e));
}

__device__ double block_sum(double v) {
  __shared__ double red[NT / 64];
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0) red[w] = v;
  __syncthreads();
  double s = 0.0;
  for (int i = 0; i < NT / 64; ++i) s += red[i];
  return s;
}

// Sum of np partials in a fixed order, by the whole workgroup.
__device__ double sum_parts(const double* part, int np) {
  double s = 0.0;
  for (int i = threadIdx.x; i < np; i += NT) s += part[i];
  __syncthreads();
  return block_sum(s);
}

__global__ __launch_bounds__(NT) void k_gather(int64_t n, const int64_t* __restrict__ perm,
                                               const double* __restrict__ user,
                                               double* __restrict__ tree) {
  const int64_t i = int64_t(blockIdx.x) * NT + threadIdx.x;
  if (i < n) tree[i] = user[perm[i]];
}

__global__ __launch_bounds__(NT) void k_scatter(int64_t n, const int64_t* __restrict__ perm,
                                                const double* __restrict__ tree,
                                                double* __restrict__ user) {
  const int64_t i = int64_t(blockIdx.x) * NT + threadIdx.x;
  if (i < n) user[perm[i]] = tree[i];
}

template <typename Td, typename Ts>
__global__ __launch_bounds__(NT) void k_cast(int64_t n, const Ts* __restrict__ s, Td* __restrict__ d) {
  const int64_t i = int64_t(blockIdx.x) * NT + threadIdx.x;
  if (i < n) d[i] = Td(s[i]);
}

template <typename Tv>
__global__ __launch_bounds__(NT) void k_axpby(int64_t n, double a, const Tv* __restrict__ x,
                                              double b, Tv* __restrict__ y) {
  const int64_t i = int64_t(blockIdx.x) * NT + threadIdx.x;
  if (i < n) y[i] = Tv(a) * x[i] + (b == 0.0 ? Tv(0) : Tv(b) * y[i]);
}

// y = x and y = 0 as kernels (no memset or memcpy nodes when a cycle is
// captured into a graph).
template <typename Tv>
__global__ __launch_bounds__(NT) void k_copy(int64_t n, const Tv* __restrict__ x, Tv* __restrict__ y) {
  const int64_t i = int64_t(blockIdx.x) * NT + threadIdx.x;
  if (i < n) y[i] = x[i];
}

template <typename Tv>
__global__ __launch_bounds__(NT) void k_zero(int64_t n, Tv* __restrict__ y) {
  const int64_t i = int64_t(blockIdx.x) * NT + threadIdx.x;
  if (i < n) y[i] = Tv(0);
}

// ---------------------------------------------------------------- gradient helpers
// user[perm[i]] = tree[i] for rows of dim coordinates.
__global__ __launch_bounds__(NT) void k_scatter_rows(int64_t n, int dim, const int64_t* __restrict__ perm,
                                                     const double* __restrict__ tree,
                                                     double* __restrict__ user) {
  const int64_t i = int64_t(blockIdx.x) * NT + threadIdx.x;
  if (i < n)
    for (int a = 0; a < dim; ++a) user[perm[i] * dim + a] = tree[i * dim + a];
}

// w_i = x_i * p_{i,a} (tree order).
__global__ __launch_bounds__(NT) void k_coord_mul(int64_t n, int dim, int a, const double* __restrict__ x,
                                                  const double* __restrict__ pts, double* __restrict__ w) {
  const int64_t i = int64_t(blockIdx.x) * NT + threadIdx.x;
  if (i < n) w[i] = x[i] * pts[i * dim + a];
}

// grad[perm[i], a] = -2 scale x_i (p_{i,a} v_i - u_i), v = G x, u = G (x * p_.a).
__global__ __launch_bounds__(NT) void k_coord_grad(int64_t n, int dim, int a, double scale,
                                                   const int64_t* __restrict__ perm,
                                                   const double* __restrict__ x,
                                                   const double* __restrict__ pts,
                                                   const double* __restrict__ v,
                                                   const double* __restrict__ u,
                                                   double* __restrict__ grad) {
  const int64_t i = int64_t(blockIdx.x) * NT + threadIdx.x;
  if (i < n) grad[perm[i] * dim + a] = -2.0 * scale * x[i] * (pts[i * dim + a] * v[i] - u[i]);
}

template <typename Tv>
__global__ __launch_bounds__(NT) void k_dot(int64_t n, const Tv* __restrict__ x,
                                            const Tv* __restrict__ y, double* __restrict__ part) {
  double acc = 0.0;
  for (int64_t i = int64_t(blockIdx.x) * NT + threadIdx.x; i < n; i += int64_t(gridDim.x) * NT)
    acc += double(x[i]) * double(y[i]);
  const double s = block_sum(acc);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// alpha = gamma / delta; e += alpha p (e = alpha p when e_zero); s -= alpha q;
// partials of s.s.  p may be s.  gamma == 0 (exact convergence) gives alpha =
// 0; delta <= 0 with gamma > 0 flags a non-SPD operator and freezes the
// iterate.
template <typename Tv>
__global__ __launch_bounds__(NT) void k_cg_update(int64_t n, Tv* __restrict__ e, bool e_zero, const Tv* p, Tv* s,
                                                  const Tv* __restrict__ q,
                                                  const double* __restrict__ gpart, int ngp,
                                                  const double* __restrict__ dpart, int ndp,
                                                  double* __restrict__ gnew, int* __restrict__ flag) {
  const double gamma = sum_parts(gpart, ngp);
  const double delta = sum_parts(dpart, ndp);
  double alpha = 0.0;
  if (gamma != 0.0) {
    if (delta > 0.0) {
      alpha = gamma / delta;
    } else if (blockIdx.x == 0 && threadIdx.x == 0) {
      atomicOr(flag, 1);
    }
  }
  double acc = 0.0;
  const Tv al = Tv(alpha);
  for (int64_t i = int64_t(blockIdx.x) * NT + threadIdx.x; i < n; i += int64_t(gridDim.x) * NT) {
    const Tv pi = p[i];
    e[i] = e_zero ? al * pi : e[i] + al * pi;
    const Tv sn = s[i] - al * q[i];
    s[i] = sn;
    acc += double(sn) * double(sn);
  }
  __syncthreads();
  const double t = block_sum(acc);
  if (threadIdx.x == 0) gnew[blockIdx.x] = t;
}

template <typename Tv>
__global__ __launch_bounds__(NT) void k_copy_dot(int64_t n, const Tv* __restrict__ src, Tv* __restrict__ s,
                                                 double* __restrict__ part) {
  double acc = 0.0;
  for (int64_t i = int64_t(blockIdx.x) * NT + threadIdx.x; i < n; i += int64_t(gridDim.x) * NT) {
    const Tv v = src[i];
    s[i] = v;
    acc += double(v) * double(v);
  }
  const double t = block_sum(acc);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// beta = gamma_new / gamma_old; p = s + beta p.
template <typename Tv>
__global__ __launch_bounds__(NT) void k_cg_pupdate(int64_t n, Tv* __restrict__ p,
                                                   const Tv* __restrict__ s,
                                                   const double* __restrict__ gold,
                                                   const double* __restrict__ gnew, int np) {
  const double go = sum_parts(gold, np);
  const double gn = sum_parts(gnew, np);
  const Tv beta = Tv(go == 0.0 ? 0.0 : gn / go);
  for (int64_t i = int64_t(blockIdx.x) * NT + threadIdx.x; i < n; i += int64_t(gridDim.x) * NT)
    p[i] = s[i] + beta * p[i];
}

template <typename Tv>
__global__ __launch_bounds__(NT) void k_check_finite(int64_t n, const Tv* __restrict__ x,
                                                     int* __restrict__ flag) {
  const int64_t i = int64_t(blockIdx.x) * NT + threadIdx.x;
  if (i < n && !isfinite(double(x[i]))) atomicOr(flag, 1);
}

// ------------------------------------------------------------ triangular solves
constexpr int NB = 64;

// x_k = L_kk^{-1} x_k (one wave).
__global__ __launch_bounds__(64) void k_trsv_fwd_diag(const double* __restrict__ L, int64_t N,
                                                      int64_t k0, double* __restrict__ x) {
  __shared__ double D[NB][NB + 1];
  const int nb = int(min<int64_t>(NB, N - k0));
  const int i = threadIdx.x;
  for (int idx = i; idx < nb * nb; idx += 64) D[idx % nb][idx / nb] = L[(k0 + idx % nb) + (k0 + idx / nb) * N];
  __syncthreads();
  double xi = i < nb ? x[k0 + i] : 0.0;
  for (int c = 0; c < nb; ++c) {
    const double xc = __shfl(xi, c, 64) / D[c][c];
    if (i == c) xi = xc;
    else if (i > c) xi -= D[i][c] * xc;
  }
  if (i < nb) x[k0 + i] = xi;
}

// x_i -= L_ik x_k for rows below block k.
__global__ __launch_bounds__(NT) void k_gemv_fwd(const double* __restrict__ L, int64_t N, int64_t k0,
                                                 double* __restrict__ x) {
  __shared__ double xk[NB];
  const int nb = int(min<int64_t>(NB, N - k0));
  if (threadIdx.x < nb) xk[threadIdx.x] = x[k0 + threadIdx.x];
  __syncthreads();
  const int64_t row = k0 + nb + int64_t(blockIdx.x) * NT + threadIdx.x;
  if (row >= N) return;
  double s = 0.0;
  for (int c = 0; c < nb; ++c) s += L[row + (k0 + c) * N] * xk[c];
  x[row] -= s;
}

// x_k = L_kk^{-T} x_k (one wave).
__global__ __launch_bounds__(64) void k_trsv_bwd_diag(const double* __restrict__ L, int64_t N,
                                                      int64_t k0, double* __restrict__ x) {
  __shared__ double D[NB][NB + 1];
  const int nb = int(min<int64_t>(NB, N - k0));
  const int i = threadIdx.x;
  for (int idx = i; idx < nb * nb; idx += 64) D[idx % nb][idx / nb] = L[(k0 + idx % nb) + (k0 + idx / nb) * N];
  __syncthreads();
  double xi = i < nb ? x[k0 + i] : 0.0;
  for (int c = nb - 1; c >= 0; --c) {
    const double xc = __shfl(xi, c, 64) / D[c][c];
    if (i == c) xi = xc;
    else if (i < c) xi -= D[c][i] * xc;
  }
  if (i < nb) x[k0 + i] = xi;
}

// x_j -= sum_i L[k0 + i][j] x_{k0 + i} for rows j above block k.
__global__ __launch_bounds__(NT) void k_gemv_bwd(const double* __restrict__ L, int64_t N, int64_t k0,
                                                 double* __restrict__ x) {
  __shared__ double xk[NB];
  const int nb = int(min<int64_t>(NB, N - k0));
  if (threadIdx.x < nb) xk[threadIdx.x] = x[k0 + threadIdx.x];
  __syncthreads();
  const int64_t j = int64_t(blockIdx.x) * NT + threadIdx.x;
  if (j >= k0) return;
  double s = 0.0;
  const double* col = L + j * N + k0;
  for (int i = 0; i < nb; ++i) s += col[i] * xk[i];
  x[j] -= s;
}

// ------------------------------------------------------------ products with the inverse factor
// The matrices of the direct solve lie in one square S (row-major): X, the inverse
// of the Cholesky factor L, up to the diagonal, and L^T above it (the diagonal of L
// in diag).
//
// Products with X alone are not backward stable: the residual of X^T (X r) grows
// with the root of the condition number (1000 rows in tree order, Gaussian
// kernel: 260 times that of substitution at condition 6e7, 17000 at 2e12).  Each triangular solve is therefore
// corrected once with its own residual, y = X r, y += X (r - L y), which leaves
// the residual of substitution as long as the factor's condition number (the
// root of the operator's) is well below 2^53.  The square of a 4096-row operator
// (134 MB) stays in the 256 MB last-level cache through the six products of a
// solve and between cycles.  They take 16 to 27 us each, 122 us together (two
// uncorrected ones 49 us); the 256 launches of substitution steps, which they
// replace, took 5.2 ms.

// y = add + sign M x, with M = X or (FACTOR) L^T: dot products with contiguous
// parts of rows of S (add may be null or y).  One wave per row, eight loads of
// 64 entries in flight.
template <bool FACTOR, typename Tin, typename Tadd, typename Tout>
__global__ __launch_bounds__(NT) void k_tri_gemv(const double* __restrict__ S, const double* __restrict__ diag,
                                                 int64_t N, const Tin* __restrict__ x, const Tadd* add, double sign,
                                                 Tout* y) {
  const int64_t i = __builtin_amdgcn_readfirstlane(int((blockIdx.x * NT + threadIdx.x) >> 6));
  if (i >= N) return;
  const int lane = threadIdx.x & 63;
  const double* row = S + i * N;
  const int64_t j1 = FACTOR ? N : i + 1;
  int64_t j = (FACTOR ? i + 1 : 0) + lane;
  double v0 = 0.0, v1 = 0.0;
  for (; j + 7 * 64 < j1; j += 8 * 64) {
    double a[8], b[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      a[q] = row[j + q * 64];
      b[q] = double(x[j + q * 64]);
    }
#pragma unroll
    for (int q = 0; q < 8; q += 2) {
      v0 += a[q] * b[q];
      v1 += a[q + 1] * b[q + 1];
    }
  }
  for (; j < j1; j += 64) v0 += row[j] * double(x[j]);
  v0 += v1;
  for (int o = 32; o > 0; o >>= 1) v0 += __shfl_xor(v0, o, 64);
  if (lane != 0) return;
  if (FACTOR) v0 += diag[i] * double(x[i]);
  y[i] = Tout(add ? double(add[i]) + sign * v0 : v0);
}

// The same with M = X^T or (FACTOR) L: sums down the columns of S.  A workgroup
// takes 16 columns (a row's part is a cache line), each of its 16 waves 4 rows
// of 64 at a time with eight loads in flight.
constexpr int NT_COL = 1024;
template <bool FACTOR, typename Tin, typename Tadd, typename Tout>
__global__ __launch_bounds__(NT_COL) void k_tri_gemv_col(const double* __restrict__ S, const double* __restrict__ diag,
                                                         int64_t N, const Tin* __restrict__ x, const Tadd* add,
                                                         double sign, Tout* y) {
  __shared__ double red[NT_COL / 64][16];
  const int p = threadIdx.x & 15;
  const int64_t c0 = int64_t(blockIdx.x) * 16, c = c0 + p, col = min(c, N - 1);
  const int64_t r1 = FACTOR ? min(N, c0 + 16) : N;
  double v = 0.0;
  for (int64_t j0 = (FACTOR ? 0 : c0) + (threadIdx.x >> 4); j0 < r1; j0 += 8 * (NT_COL / 16)) {
    double a[8], b[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int64_t j = j0 + q * (NT_COL / 16);
      const bool in = j < r1 && (FACTOR ? j < c : j >= c);
      a[q] = in ? S[j * N + col] : 0.0;
      b[q] = in ? double(x[j]) : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) v += a[q] * b[q];
  }
  v += __shfl_xor(v, 16, 64);
  v += __shfl_xor(v, 32, 64);
  if ((threadIdx.x & 63) < 16) red[threadIdx.x >> 6][p] = v;
  __syncthreads();
  if (threadIdx.x >= 16 || c >= N) return;
  v = 0.0;
  for (int w = 0; w < NT_COL / 64; ++w) v += red[w][p];
  if (FACTOR) v += diag[c] * double(x[c]);
  y[c] = Tout(add ? double(add[c]) + sign * v : v);
}

inline unsigned blocks(int64_t n) { return unsigned((n + NT - 1) / NT); }

}  // namespace

int dot_parts(int64_t n) {
  return int(std::max<int64_t>(1, std::min<int64_t>(MAX_PARTS, (n + 4095) / 4096)));
}

void launch_gather(H2& h, const double* user, double* tree) {
  hipLaunchKernelGGL(k_gather, dim3(blocks(h.n)), dim3(NT), 0, h.stream, int64_t(h.n), h.perm, user, tree);
  check_launch("gather");
}

void launch_scatter(H2& h, const double* tree, double* user) {
  hipLaunchKernelGGL(k_scatter, dim3(blocks(h.n)), dim3(NT), 0, h.stream, int64_t(h.n), h.perm, tree, user);
  check_launch("scatter");
}

void launch_copy(H2& h, int p, const void* src, void* dst, int64_t n) {
  if (n <= 0) return;
  if (p == P64)
    hipLaunchKernelGGL(k_copy<double>, dim3(blocks(n)), dim3(NT), 0, h.stream, n,
                       static_cast<const double*>(src), static_cast<double*>(dst));
  else
    hipLaunchKernelGGL(k_copy<float>, dim3(blocks(n)), dim3(NT), 0, h.stream, n,
                       static_cast<const float*>(src), static_cast<float*>(dst));
  check_launch("copy");
}

void launch_zero(H2& h, int p, void* dst, int64_t n) {
  if (n <= 0) return;
  if (p == P64)
    hipLaunchKernelGGL(k_zero<double>, dim3(blocks(n)), dim3(NT), 0, h.stream, n, static_cast<double*>(dst));
  else
    hipLaunchKernelGGL(k_zero<float>, dim3(blocks(n)), dim3(NT), 0, h.stream, n, static_cast<float*>(dst));
  check_launch("zero");
}

void launch_cast(H2& h, int pdst, void* dst, int psrc, const void* src, int64_t n) {
  const bool d64 = pdst == P64, s64 = psrc == P64;
  if (d64 == s64) { launch_copy(h, pdst, src, dst, n); return; }
  if (d64)
    hipLaunchKernelGGL((k_cast<double, float>), dim3(blocks(n)), dim3(NT), 0, h.stream, n,
                       static_cast<const float*>(src), static_cast<double*>(dst));
  else
    hipLaunchKernelGGL((k_cast<float, double>), dim3(blocks(n)), dim3(NT), 0, h.stream, n,
                       static_cast<const double*>(src), static_cast<float*>(dst));
  check_launch("cast");
}

void launch_axpby(H2& h, int p, int64_t n, double a, const void* x, double b, void* y) {
  if (p == P64)
    hipLaunchKernelGGL(k_axpby<double>, dim3(blocks(n)), dim3(NT), 0, h.stream, n, a,
                       static_cast<const double*>(x), b, static_cast<double*>(y));
  else
    hipLaunchKernelGGL(k_axpby<float>, dim3(blocks(n)), dim3(NT), 0, h.stream, n, a,
                       static_cast<const float*>(x), b, static_cast<float*>(y));
  check_launch("axpby");
}

void launch_dot(H2& h, int p, int64_t n, const void* x, const void* y, double* part) {
  const int np = dot_parts(n);
  if (p == P64)
    hipLaunchKernelGGL(k_dot<double>, dim3(np), dim3(NT), 0, h.stream, n,
                       static_cast<const double*>(x), static_cast<const double*>(y), part);
  else
    hipLaunchKernelGGL(k_dot<float>, dim3(np), dim3(NT), 0, h.stream, n,
                       static_cast<const float*>(x), static_cast<const float*>(y), part);
  check_launch("dot");
}

void launch_cg_update(H2& h, int p, int64_t n, void* e, bool e_zero, const void* pv, void* s, const void* q,
                      const double* gamma_part, int ngp, const double* delta_part, int ndp,
                      double* gamma_new_part) {
  const int np = dot_parts(n);
  if (p == P64)
    hipLaunchKernelGGL(k_cg_update<double>, dim3(np), dim3(NT), 0, h.stream, n,
                       static_cast<double*>(e), e_zero, static_cast<const double*>(pv),
                       static_cast<double*>(s), static_cast<const double*>(q), gamma_part, ngp,
                       delta_part, ndp, gamma_new_part, h.flags);
  else
    hipLaunchKernelGGL(k_cg_update<float>, dim3(np), dim3(NT), 0, h.stream, n,
                       static_cast<float*>(e), e_zero, static_cast<const float*>(pv),
                       static_cast<float*>(s), static_cast<const float*>(q), gamma_part, ngp,
                       delta_part, ndp, gamma_new_part, h.flags);
  check_launch("cg_update");
}

void launch_cg_pupdate(H2& h, int p, int64_t n, void* pv, const void* s,
                       const double* gamma_old_part, const double* gamma_new_part, int np) {
  const dim3 g(dot_parts(n)), b(NT);
  if (p == P64)
    hipLaunchKernelGGL(k_cg_pupdate<double>, g, b, 0, h.stream, n,
                       static_cast<double*>(pv), static_cast<const double*>(s), gamma_old_part,
                       gamma_new_part, np);
  else
    hipLaunchKernelGGL(k_cg_pupdate<float>, g, b, 0, h.stream, n,
                       static_cast<float*>(pv), static_cast<const float*>(s), gamma_old_part,
                       gamma_new_part, np);
  check_launch("cg_pupdate");
}

void launch_copy_dot(H2& h, int p, int64_t n, const void* src, void* s, double* part) {
  const dim3 g(dot_parts(n)), b(NT);
  if (p == P64)
    hipLaunchKernelGGL(k_copy_dot<double>, g, b, 0, h.stream, n, static_cast<const double*>(src),
                       static_cast<double*>(s), part);
  else
    hipLaunchKernelGGL(k_copy_dot<float>, g, b, 0, h.stream, n, static_cast<const float*>(src),
                       static_cast<float*>(s), part);
  check_launch("copy_dot");
}

void launch_chol_solve(H2& h, const double* L, int64_t N, double* x) {
  for (int64_t k0 = 0; k0 < N; k0 += NB) {
    hipLaunchKernelGGL(k_trsv_fwd_diag, dim3(1), dim3(64), 0, h.stream, L, N, k0, x);
    const int64_t below = N - k0 - std::min<int64_t>(NB, N - k0);
    if (below > 0)
      hipLaunchKernelGGL(k_gemv_fwd, dim3(blocks(below)), dim3(NT), 0, h.stream, L, N, k0, x);
  }
  const int64_t last = ((N - 1) / NB) * NB;
  for (int64_t k0 = last; k0 >= 0; k0 -= NB) {
    hipLaunchKernelGGL(k_trsv_bwd_diag, dim3(1), dim3(64), 0, h.stream, L, N, k0, x);
    if (k0 > 0)
      hipLaunchKernelGGL(k_gemv_bwd, dim3(blocks(k0)), dim3(NT), 0, h.stream, L, N, k0, x);
  }
  check_launch("chol_solve");
}

void launch_inverse_solve(H2& h, int p, const void* r, void* e) {
  const int64_t N = h.Nl;
  const dim3 g(unsigned((N + NT / 64 - 1) / (NT / 64))), b(NT), gc(unsigned((N + 15) / 16)), bc(NT_COL);
  const double *S = h.cinv, *d = h.cdiag, *none = nullptr;
  double *y = h.vtree2, *t = h.vtree;
  auto solve = [&](auto tv) {
    using Tv = decltype(tv);
    const Tv* rv = static_cast<const Tv*>(r);
    hipLaunchKernelGGL((k_tri_gemv<false, Tv, double, double>), g, b, 0, h.stream, S, d, N, rv, none, 1.0, y);
    hipLaunchKernelGGL((k_tri_gemv_col<true, double, Tv, double>), gc, bc, 0, h.stream, S, d, N, y, rv, -1.0, t);
    hipLaunchKernelGGL((k_tri_gemv<false, double, double, double>), g, b, 0, h.stream, S, d, N, t, y, 1.0, y);
    hipLaunchKernelGGL((k_tri_gemv_col<false, double, double, double>), gc, bc, 0, h.stream, S, d, N, y, none, 1.0, t);
    hipLaunchKernelGGL((k_tri_gemv<true, double, double, double>), g, b, 0, h.stream, S, d, N, t, y, -1.0, y);
    hipLaunchKernelGGL((k_tri_gemv_col<false, double, double, Tv>), gc, bc, 0, h.stream, S, d, N, y, t, 1.0,
                       static_cast<Tv*>(e));
  };
  if (p == P64) solve(double{});
  else solve(float{});
  check_launch("inverse_solve");
}

void launch_scatter_rows(H2& h, const double* tree, double* user) {
  hipLaunchKernelGGL(k_scatter_rows, dim3(blocks(h.n)), dim3(NT), 0, h.stream, int64_t(h.n), h.dim,
                     h.perm, tree, user);
  check_launch("scatter_rows");
}

void launch_coord_mul(H2& h, int a, const double* x, double* w) {
  hipLaunchKernelGGL(k_coord_mul, dim3(blocks(h.n)), dim3(NT), 0, h.stream, int64_t(h.n), h.dim, a, x,
                     h.pts, w);
  check_launch("coord_mul");
}

void launch_coord_grad(H2& h, int a, double scale, const double* x, const double* v, const double* u,
                       double* grad) {
  hipLaunchKernelGGL(k_coord_grad, dim3(blocks(h.n)), dim3(NT), 0, h.stream, int64_t(h.n), h.dim, a,
                     scale, h.perm, x, h.pts, v, u, grad);
  check_launch("coord_grad");
}

void launch_check_finite(H2& h, int p, int64_t n, const void* x) {
  if (p == P64)
    hipLaunchKernelGGL(k_check_finite<double>, dim3(blocks(n)), dim3(NT), 0, h.stream, n,
                       static_cast<const double*>(x), h.flags + 1);
  else
    hipLaunchKernelGGL(k_check_finite<float>, dim3(blocks(n)), dim3(NT), 0, h.stream, n,
                       static_cast<const float*>(x), h.flags + 1);
  check_launch("check_finite");
}

}  // namespace h2mg
