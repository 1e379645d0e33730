// The sweeps over the cluster tree (Section 3.1: x_{d-1} = E^T x_d upwards,
// y_d += E y_{d-1} downwards) with several levels in one launch, and the steps
// of the CG smoother that ride on them.
//
// A level of a sweep moves little (one transfer tile per cluster, 0.3 to 30 us
// worth of bandwidth over all levels), so with one launch per level its cost
// was the launches: 3 to 9 us each, a fifth of a solve on 65536 points.  Here
// a workgroup takes a whole subtree of `nlev` levels below its root cluster,
// with the coefficients of the current level in LDS: no workgroup waits for
// another one.  A wave takes one child tile (the 64-lane layout of
// device_common.h), small tiles several at a time so that enough loads are in
// flight.  A sweep of two or three levels takes 6 us in FP32, one of four
// levels 11 us in FP64 (4.5 and 6 to 9 us a level before); with the steps
// below a CG step is 5 launches instead of 10 to 16, and the solve went from
// 397 to 302 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <stdexcept>
#include <string>

#include "h2_impl.h"

namespace h2mg {

namespace {

void check_launch(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) throw std::runtime_error(std::string(what) + ": " + hipGetErrorString(e));
}

// Threads of a workgroup: a 64 x 64 FP64 tile takes 128 registers per lane,
// so those run with eight waves, smaller ones with sixteen.  Tiles a wave
// holds at once: 64 elements per lane.
template <int T> constexpr int SWEEP_NT = T == 8 ? 512 : 1024;
template <int T> constexpr int SWEEP_UNROLL = T == 8 ? 1 : T == 4 ? 2 : 8;
// Levels per launch: up to half a megabyte of FP64 tiles per workgroup, and at
// most 1024 coefficients a level.  Four levels of 64 x 64 tiles in one launch
// (a megabyte for each of 64 workgroups) took 27 us up and 22 us down, two and
// two of them 21 and 22 us (100k points).
constexpr int sweep_levels(int T) { return T == 8 ? 3 : T == 4 ? 4 : 6; }
constexpr int SWEEP_BUF = 1024;        // coefficients of one level of a subtree: 2^nlev * r at most

// Sum of np partial sums by the whole workgroup, in a fixed order.
template <int NT>
__device__ inline double parts_sum(const double* part, int np, double* red) {
  double s = 0.0;
  for (int i = threadIdx.x; i < np; i += NT) s += part[i];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  s = 0.0;
  for (int i = 0; i < NT / 64; ++i) s += red[i];
  return s;
}

// Upwards from depth d = q + nlev to depth q; workgroup b: the subtree of
// cluster b of depth q.  xall: coefficients of every cluster by gid.  The
// coefficients of depth d are
//   * those in xall (src null),
//   * src, copied there (zd null), or
//   * the next CG direction p = src + beta zd (zd: the direction before, which
//     may be the place in xall itself), beta = sum(gnew) / sum(gold).
template <int T, typename Tb, typename Tv>
__global__ __launch_bounds__(SWEEP_NT<T>) void k_sweep_up(int q, int nlev, int r, const Tb* __restrict__ E,
                                                          Tv* xall, const Tv* src, const Tv* zd,
                                                          const double* __restrict__ gold,
                                                          const double* __restrict__ gnew, int np) {
  constexpr int NT = SWEEP_NT<T>, U = SWEEP_UNROLL<T>;
  __shared__ Tv cur[SWEEP_BUF], tmp[SWEEP_BUF];
  __shared__ double red[NT / 64];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int a = lane >> 3, b = lane & 7;
  const int d = q + nlev;
  const int64_t g0 = (int64_t(1) << d) - 1 + (int64_t(blockIdx.x) << nlev);   // first gid of depth d here
  Tv beta = Tv(0);
  if (zd) {
    const double go = parts_sum<NT>(gold, np, red), gn = parts_sum<NT>(gnew, np, red);
    beta = Tv(go == 0.0 ? 0.0 : gn / go);
  }
  Tv* xd = xall + g0 * r;
  const int64_t off = int64_t(blockIdx.x) * (r << nlev);    // first coefficient among those of depth d
  for (int i = tid; i < r << nlev; i += NT) {
    Tv v;
    if (src) {
      v = zd ? src[off + i] + beta * zd[off + i] : src[off + i];
      xd[i] = v;
    } else {
      v = xd[i];
    }
    cur[i] = v;
  }
  __syncthreads();
  for (int l = nlev; l > 0; --l) {
    const int nc = 1 << l;             // children here at relative depth l
    const int64_t gc = (int64_t(1) << (q + l)) - 1 + (int64_t(blockIdx.x) << l);
    for (int c0 = w * U; c0 < nc; c0 += NT / 64 * U) {
      Tv B[U][T * T];
#pragma unroll
      for (int k = 0; k < U; ++k)
        if (c0 + k < nc) load_subtile<T, Tb, Tv>(E + (gc + c0 + k) * tile_elems(T), lane, tile_A(r, T), B[k]);
#pragma unroll
      for (int k = 0; k < U; ++k) {
        if (c0 + k >= nc) break;
        Tv z[T];
#pragma unroll
        for (int v = 0; v < T; ++v) z[v] = Tv(0);
#pragma unroll
        for (int u = 0; u < T; ++u) {
          const int i = a * T + u;
          const Tv xs = i < r ? cur[(c0 + k) * r + i] : Tv(0);
#pragma unroll
          for (int v = 0; v < T; ++v) z[v] += B[k][u * T + v] * xs;
        }
        const Tv s = transpose_reduce_a<T, Tv>(z, a);
        const int j = b * T + reduced_index<T>(a);
        if ((T == 8 || (a & ((8 / T) - 1)) == 0) && j < r) tmp[(c0 + k) * r + j] = s;
      }
    }
    __syncthreads();
    Tv* xp = xall + ((int64_t(1) << (q + l - 1)) - 1 + (int64_t(blockIdx.x) << (l - 1))) * r;
    for (int i = tid; i < r << (l - 1); i += NT) {
      const int s = i / r, j = i - s * r;
      const Tv v = tmp[2 * s * r + j] + tmp[(2 * s + 1) * r + j];
      cur[i] = v;
      xp[i] = v;
    }
    __syncthreads();
  }
}

// Downwards from depth q to depth d = q + nlev: y_c = yall[c] + E_c y_parent
// within the subtree of cluster b of depth q.  out (d's coefficients, may be
// d's place in yall) = y_d, or add - y_d when add is given; with dpart, the
// partial sums of out . xd (xd: depth d's coefficients of another vector).
template <int T, typename Tb, typename Tv>
__global__ __launch_bounds__(SWEEP_NT<T>) void k_sweep_down(int q, int nlev, int r, const Tb* __restrict__ E,
                                                            const Tv* yall, Tv* out, const Tv* add, const Tv* xd,
                                                            double* __restrict__ dpart) {
  constexpr int NT = SWEEP_NT<T>, U = SWEEP_UNROLL<T>;
  __shared__ Tv par[SWEEP_BUF / 2], cur[SWEEP_BUF];
  __shared__ double red[NT / 64];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int a = lane >> 3, b = lane & 7;
  const Tv* yq = yall + ((int64_t(1) << q) - 1 + blockIdx.x) * r;
  for (int i = tid; i < r; i += NT) par[i] = yq[i];
  for (int l = 1; l <= nlev; ++l) {
    const int nc = 1 << l;
    const int64_t gc = (int64_t(1) << (q + l)) - 1 + (int64_t(blockIdx.x) << l);
    const Tv* yl = yall + gc * r;
    for (int i = tid; i < r << l; i += NT) cur[i] = yl[i];
    __syncthreads();
    for (int c0 = w * U; c0 < nc; c0 += NT / 64 * U) {
      Tv B[U][T * T];
#pragma unroll
      for (int k = 0; k < U; ++k)
        if (c0 + k < nc) load_subtile<T, Tb, Tv>(E + (gc + c0 + k) * tile_elems(T), lane, tile_A(r, T), B[k]);
#pragma unroll
      for (int k = 0; k < U; ++k) {
        if (c0 + k >= nc) break;
        const int s = (c0 + k) >> 1;
        Tv z[T];
#pragma unroll
        for (int u = 0; u < T; ++u) z[u] = Tv(0);
#pragma unroll
        for (int v = 0; v < T; ++v) {
          const int j = b * T + v;
          const Tv xt = j < r ? par[s * r + j] : Tv(0);
#pragma unroll
          for (int u = 0; u < T; ++u) z[u] += B[k][u * T + v] * xt;
        }
#pragma unroll
        for (int u = 0; u < T; ++u) {
          Tv v = z[u];
          v += shfl_xor(v, 1);
          v += shfl_xor(v, 2);
          v += shfl_xor(v, 4);
          z[u] = v;
        }
        if (b == 0) {
#pragma unroll
          for (int u = 0; u < T; ++u)
            if (a * T + u < r) cur[(c0 + k) * r + a * T + u] += z[u];
        }
      }
    }
    __syncthreads();
    if (l < nlev) {
      for (int i = tid; i < r << l; i += NT) par[i] = cur[i];
      __syncthreads();
    }
  }
  const int64_t off = int64_t(blockIdx.x) * (r << nlev);
  double acc = 0.0;
  for (int i = tid; i < r << nlev; i += NT) {
    const Tv v = add ? Tv(-1) * cur[i] + add[off + i] : cur[i];
    out[off + i] = v;
    if (dpart) acc += double(v) * double(xd[off + i]);
  }
  if (dpart) {
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if (lane == 0) red[w] = acc;
    __syncthreads();
    if (tid == 0) {
      double s = 0.0;
      for (int i = 0; i < NT / 64; ++i) s += red[i];
      dpart[blockIdx.x] = s;
    }
  }
}

// ------------------------------------------------------------ CG steps
// alpha = gamma / delta; e += alpha p (e = alpha p when e_zero); s -= alpha q;
// z = M^{-1} s on the diagonal blocks (rows [off[b], off[b+1]), or
// [b * stride, (b+1) * stride)); partial sums of s . z.  Without p: z and the
// sums of the given s only.  gamma == 0 (exact convergence) gives alpha = 0;
// delta <= 0 with gamma > 0 flags a non-SPD operator and freezes the iterate.
// A block's rows belong to one workgroup, so the update, the block product
// and the dot product need one pass and one launch instead of three.  The
// inverses are symmetric: thread (i, g) sums the g-th part of column i.
template <typename Tv>
__global__ __launch_bounds__(256) void k_cg_step_bj(int nblocks, const int* __restrict__ off, int stride,
                                                    const Tv* __restrict__ Minv, int ld, const Tv* src, Tv* e,
                                                    bool e_zero, const Tv* p, Tv* s, const Tv* q, Tv* z,
                                                    const double* __restrict__ gpart, int ngp,
                                                    const double* __restrict__ dpart, int ndp,
                                                    double* __restrict__ gnew, int* __restrict__ flag) {
  __shared__ Tv sl[128];
  __shared__ Tv part[256];
  __shared__ double red[4];
  const int tid = threadIdx.x;
  Tv al = Tv(0);
  if (p) {
    const double gamma = parts_sum<256>(gpart, ngp, red), delta = parts_sum<256>(dpart, ndp, red);
    double alpha = 0.0;
    if (gamma != 0.0) {
      if (delta > 0.0) alpha = gamma / delta;
      else if (blockIdx.x == 0 && tid == 0) atomicOr(flag, 1);
    }
    al = Tv(alpha);
  }
  double acc = 0.0;
  for (int b = blockIdx.x; b < nblocks; b += gridDim.x) {
    const int s0 = off ? off[b] : b * stride;
    const int n = off ? off[b + 1] - s0 : stride;
    const int np = n <= 32 ? 32 : n <= 64 ? 64 : 128, ng = 256 / np;
    __syncthreads();
    if (tid < n) {
      const int64_t i = s0 + tid;
      Tv sn;
      if (p) {
        e[i] = e_zero ? al * p[i] : e[i] + al * p[i];
        sn = s[i] - al * q[i];
      } else {
        sn = src[i];
      }
      s[i] = sn;
      sl[tid] = sn;
    }
    __syncthreads();
    const int i = tid & (np - 1), g = tid / np;
    Tv v = Tv(0);
    if (i < n) {
      const Tv* M = Minv + int64_t(b) * ld * ld + i;
      const int j1 = (g + 1) * n / ng;
#pragma unroll 8
      for (int j = g * n / ng; j < j1; ++j) v += M[int64_t(j) * ld] * sl[j];
    }
    part[tid] = v;
    __syncthreads();
    if (tid < n) {
      Tv t = part[tid];
      for (int k = 1; k < ng; ++k) t += part[k * np + tid];
      z[s0 + tid] = t;
      acc += double(sl[tid]) * double(t);
    }
  }
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  __syncthreads();
  if ((tid & 63) == 0) red[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) gnew[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

template <typename F>
void dispatch_T(int T, F&& f) {
  switch (T) {
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    default: f(std::integral_constant<int, 8>{}); break;
  }
}

// f(Tv{}, Tb{}) for an operator precision.
template <typename F>
void dispatch_prec(int p, F&& f) {
  if (p == P64) f(double{}, double{});
  else if (p == P32) f(float{}, float{});
  else f(float{}, bf16{});
}

// Levels of the launch that covers depths (q, d]: all of them when they fit,
// else equal shares.
int levels_of(int n, int T) {
  const int k = sweep_levels(T), launches = (n + k - 1) / k;
  return (n + launches - 1) / launches;
}

}  // namespace

void launch_sweep_up(H2& h, int p, int d, void* xall, const void* src, const void* zd, const double* gold,
                     const double* gnew, int np) {
  bool first = true;
  for (int top = d; top > h.d_top || first;) {
    const int nlev = std::min(levels_of(std::max(d - h.d_top, 1), h.T), top - h.d_top);
    const int q = top - nlev;
    dispatch_T(h.T, [&](auto Tc) {
      constexpr int T = decltype(Tc)::value;
      dispatch_prec(p, [&](auto tv, auto tb) {
        using Tv = decltype(tv);
        using Tb = decltype(tb);
        hipLaunchKernelGGL((k_sweep_up<T, Tb, Tv>), dim3(1u << q), dim3(SWEEP_NT<T>), 0, h.stream, q, nlev, h.r,
                           static_cast<const Tb*>(h.prec[p].E), static_cast<Tv*>(xall),
                           static_cast<const Tv*>(first ? src : nullptr), static_cast<const Tv*>(first ? zd : nullptr),
                           gold, gnew, np);
      });
    });
    top = q;
    first = false;
  }
  check_launch("sweep_up");
}

int launch_sweep_down(H2& h, int p, int d, void* yall, void* out, const void* add, const void* xd,
                      double* dpart) {
  const int share = levels_of(std::max(d - h.d_top, 1), h.T);
  int blocks = 0;
  // the last launch ends at depth d; the ones before write into yall
  for (int q = h.d_top; q < d;) {
    int nlev = (d - q) % share;
    if (nlev == 0) nlev = share;
    const bool last = q + nlev == d;
    dispatch_T(h.T, [&](auto Tc) {
      constexpr int T = decltype(Tc)::value;
      dispatch_prec(p, [&](auto tv, auto tb) {
        using Tv = decltype(tv);
        using Tb = decltype(tb);
        Tv* y = static_cast<Tv*>(yall);
        Tv* mid = y + ((int64_t(1) << (q + nlev)) - 1) * h.r;
        hipLaunchKernelGGL((k_sweep_down<T, Tb, Tv>), dim3(1u << q), dim3(SWEEP_NT<T>), 0, h.stream, q, nlev, h.r,
                           static_cast<const Tb*>(h.prec[p].E), y, last ? static_cast<Tv*>(out) : mid,
                           static_cast<const Tv*>(last ? add : nullptr), static_cast<const Tv*>(xd),
                           last ? dpart : nullptr);
      });
    });
    blocks = 1 << q;
    q += nlev;
  }
  check_launch("sweep_down");
  return blocks;
}

int launch_cg_step_bj(H2& h, int p, int k, const void* src, void* e, bool e_zero, const void* pv, void* s,
                      const void* q, void* z, const double* gpart, int ngp, const double* dpart, int ndp, double* gnew) {
  const bool fine = k == 1;
  const int d = h.level_depth(k);
  const int nb = fine ? h.nleaf : (1 << d);
  const int* off = fine ? h.leaf_off : nullptr;
  const int ld = fine ? h.bj_ld : h.r;
  const int grid = std::min(nb, DOT_PARTS);
  dispatch_prec(p, [&](auto tv, auto) {
    using Tv = decltype(tv);
    const int pp = p == P64 ? P64 : P32;
    const Tv* M = static_cast<const Tv*>(fine ? h.bj_fine[pp] : h.bj_coarse[pp]);
    if (!fine) M += ((int64_t(1) << d) - 1) * h.r * h.r;
    hipLaunchKernelGGL((k_cg_step_bj<Tv>), dim3(grid), dim3(256), 0, h.stream, nb, off, h.r, M, ld,
                       static_cast<const Tv*>(src), static_cast<Tv*>(e), e_zero, static_cast<const Tv*>(pv), static_cast<Tv*>(s),
                       static_cast<const Tv*>(q), static_cast<Tv*>(z), gpart, ngp, dpart, ndp, gnew, h.flags);
  });
  check_launch("cg_step_bj");
  return grid;
}

}  // namespace h2mg
