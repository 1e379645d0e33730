// The tree sweeps on blocks of 16 vectors with several levels in one launch,
// the block-Jacobi CG step on such blocks, and the products with the leaf
// bases, all on the matrix cores (see kernels_sweep.hip for the single-vector
// forms, kernels_block.hip for the block layout: entry (i, k) at i * 16 + k).
//
// Lane (p, q) = (lane % 16, lane / 16) supplies A[p][q] and B[q][p] of a
// 16 x 16 x 4 product; result element t is row M::row(t, q), column p.  A wave
// takes a slab of 16 result rows of one cluster.  The A operands (transfers,
// inverses, bases) are read straight from memory: each is used once per
// launch, and the 16 lanes of a row read 64 to 128 consecutive bytes or, in
// the tile layout, pieces that the next steps complete; staging them in LDS,
// one tile per workgroup and launch, made every level of a sweep a launch of
// its own (4 us each, a fifth of a 16-column solve on 16500 points, which went
// from 133 to 122 ms).  The leaf products on 65536 points take 12 and 15 us
// instead of 141 and 117 with one entry per thread.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <stdexcept>
#include <string>
#include <type_traits>

#include "h2_impl.h"

namespace h2mg {

namespace {

constexpr int NR = MULTI_NR;
constexpr int SWEEP_NT = 512;

void check_launch(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) throw std::runtime_error(std::string(what) + ": " + hipGetErrorString(e));
}

// sums[k] = sum over b < np of part[b * 16 + k] by a workgroup of N threads,
// in a fixed order (red: N doubles).  Eight loads in flight: one at a time,
// the 512 sums of a step were a chain of 16 memory latencies in every
// workgroup of the next kernel (a 16-column solve of 16k points: 105 ms, now
// 99 ms).
template <int N>
__device__ inline void colsum(const double* __restrict__ part, int np, double* sums, double* red) {
  const int k = threadIdx.x & 15;
  double s = 0.0;
  int b = threadIdx.x >> 4;
  for (; b + 7 * (N / 16) < np; b += 8 * (N / 16)) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = part[(b + u * (N / 16)) * NR + k];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
#pragma unroll 4
  for (; b < np; b += N / 16) s += part[b * NR + k];
  __syncthreads();
  red[threadIdx.x] = s;
  __syncthreads();
  if (threadIdx.x < NR) {
    double t = 0.0;
    for (int w = 0; w < N / 16; ++w) t += red[w * NR + threadIdx.x];
    sums[threadIdx.x] = t;
  }
  __syncthreads();
}

// part[blockIdx * 16 + p] = the sum of acc over the lanes of column p.
template <int N>
__device__ inline void colpart(double acc, double* red, double* __restrict__ part) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  acc += __shfl_xor(acc, 16, 64);
  acc += __shfl_xor(acc, 32, 64);
  __syncthreads();
  if (lane < NR) red[w * NR + lane] = acc;
  __syncthreads();
  if (threadIdx.x < NR) {
    double t = 0.0;
    for (int v = 0; v < N / 64; ++v) t += red[v * NR + threadIdx.x];
    part[blockIdx.x * NR + threadIdx.x] = t;
  }
}

// Upwards from depth d = q + nlev to depth q within the subtree of cluster
// blockIdx of depth q.  The coefficients of depth d: those in xall (src null),
// src, or src + beta prev with beta = sum(gnew) / sum(gold) per column (prev
// may be their place in xall); they are left in keep unless it is null.  Those
// of depth q go to xroot, those between into xall.
template <int T, typename Te, typename Tv>
__global__ __launch_bounds__(SWEEP_NT) void k_sweep_up16(int q0, int nlev, int r, const Te* __restrict__ E, Tv* xall,
                                                         const Tv* src, const Tv* prev, Tv* keep, Tv* xroot,
                                                         const double* __restrict__ gold,
                                                         const double* __restrict__ gnew, int np) {
  using M = Mfma<Tv>;
  constexpr int NKB = 2 * T;           // k-steps of a child tile of 8T rows
  extern __shared__ double lds_raw[];
  __shared__ double red[SWEEP_NT];
  __shared__ double go[NR], gn[NR];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, p = lane & 15, q = lane >> 4;
  const int64_t nd = int64_t(r) * NR << nlev;
  Tv* cur = reinterpret_cast<Tv*>(lds_raw);
  Tv* nxt = cur + nd;
  const Tv* xd = (src ? src : xall + ((int64_t(1) << (q0 + nlev)) - 1) * r * NR) + blockIdx.x * nd;
  Tv beta = Tv(0);
  if (prev) {
    colsum<SWEEP_NT>(gold, np, go, red);
    colsum<SWEEP_NT>(gnew, np, gn, red);
    beta = Tv(go[p] == 0.0 ? 0.0 : gn[p] / go[p]);   // column tid % 16 = p
  }
  for (int64_t i = tid; i < nd; i += SWEEP_NT) {
    Tv v = xd[i];
    if (prev) v += beta * prev[blockIdx.x * nd + i];
    if (keep) keep[blockIdx.x * nd + i] = v;
    cur[i] = v;
  }
  __syncthreads();
  const int ns = (r + 15) >> 4, A = tile_A(r, T);
  for (int l = nlev; l > 0; --l) {
    const int64_t gc = (int64_t(1) << (q0 + l)) - 1 + (int64_t(blockIdx.x) << l);
    Tv* xp = l == 1 ? xroot + int64_t(blockIdx.x) * r * NR
                    : xall + ((int64_t(1) << (q0 + l - 1)) - 1 + (int64_t(blockIdx.x) << (l - 1))) * r * NR;
    for (int it = w; it < ns << (l - 1); it += SWEEP_NT / 64) {
      const int s = it / ns, j = 16 * (it % ns) + p;
      typename M::acc_t acc = typename M::acc_t{Tv(0), Tv(0), Tv(0), Tv(0)};
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int c = 2 * s + h;
        const Te* tile = E + (gc + c) * tile_elems(T);
        Tv a[NKB];
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
          const int k = 4 * kb + q;
          a[kb] = k < r && j < r ? ld_as<Tv, Te>(tile[tile_offset<Te>(k, j, T, A)]) : Tv(0);
        }
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
          const int k = 4 * kb + q;
          if (4 * kb < r) acc = M::mma(a[kb], k < r ? cur[(c * r + k) * NR + p] : Tv(0), acc);
        }
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int row = 16 * (it % ns) + M::row(t, q);
        if (row < r) {
          nxt[(s * r + row) * NR + p] = acc[t];
          xp[(s * r + row) * NR + p] = acc[t];
        }
      }
    }
    __syncthreads();
    Tv* o = cur;
    cur = nxt;
    nxt = o;
  }
}

// Downwards from depth q to depth d = q + nlev: y_c = yall[c] + E_c y_parent,
// with y_q in root and depth d's part of yall in ybot (which may be out).
// out = y_d or add - y_d; with dpart the per-column partial sums of out . xd.
template <int T, typename Te, typename Tv>
__global__ __launch_bounds__(SWEEP_NT) void k_sweep_down16(int q0, int nlev, int r, const Te* __restrict__ E,
                                                           const Tv* yall, const Tv* root, const Tv* ybot, Tv* out,
                                                           const Tv* add, const Tv* xd, double* __restrict__ dpart) {
  using M = Mfma<Tv>;
  constexpr int NKB = 2 * T;
  extern __shared__ double lds_raw[];
  __shared__ double red[SWEEP_NT];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, p = lane & 15, q = lane >> 4;
  Tv* par = reinterpret_cast<Tv*>(lds_raw);
  Tv* cur = par + (int64_t(r) * NR << (nlev - 1));
  const Tv* yq = root + int64_t(blockIdx.x) * r * NR;
  for (int i = tid; i < r * NR; i += SWEEP_NT) par[i] = yq[i];
  __syncthreads();
  const int ns = (r + 15) >> 4, A = tile_A(r, T);
  const int64_t off = blockIdx.x * (int64_t(r) * NR << nlev);
  double dacc = 0.0;
  for (int l = 1; l <= nlev; ++l) {
    const int64_t gc = (int64_t(1) << (q0 + l)) - 1 + (int64_t(blockIdx.x) << l);
    const Tv* yl = l == nlev ? ybot + off : yall + gc * r * NR;
    for (int it = w; it < ns << l; it += SWEEP_NT / 64) {
      const int c = it / ns, s = c >> 1, i = 16 * (it % ns) + p;
      const Te* tile = E + (gc + c) * tile_elems(T);
      Tv a[NKB];
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
        const int k = 4 * kb + q;
        a[kb] = k < r && i < r ? ld_as<Tv, Te>(tile[tile_offset<Te>(i, k, T, A)]) : Tv(0);
      }
      typename M::acc_t acc;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int row = 16 * (it % ns) + M::row(t, q);
        acc[t] = row < r ? yl[(c * r + row) * NR + p] : Tv(0);
      }
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
        const int k = 4 * kb + q;
        if (4 * kb < r) acc = M::mma(a[kb], k < r ? par[(s * r + k) * NR + p] : Tv(0), acc);
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int row = 16 * (it % ns) + M::row(t, q);
        if (row >= r) continue;
        const int e = (c * r + row) * NR + p;
        if (l < nlev) {
          cur[e] = acc[t];
        } else {
          const Tv v = add ? add[off + e] - acc[t] : acc[t];
          out[off + e] = v;
          if (dpart) dacc += double(v) * double(xd[off + e]);
        }
      }
    }
    __syncthreads();
    Tv* o = par;
    par = cur;
    cur = o;
  }
  if (dpart) colpart<SWEEP_NT>(dacc, red, dpart);
}

// A step of the block-Jacobi CG on every column (see k_cg_step_bj): e += alpha
// p, s -= alpha q, z = M^{-1} s per diagonal block, partial sums of s . z;
// without p: s = src, z and the sums.
template <typename Tv>
__global__ __launch_bounds__(256) void k_cg_step16_bj(int nblocks, const int* __restrict__ off, int stride,
                                                      const Tv* __restrict__ Minv, int ld, const Tv* src, Tv* e,
                                                      bool e_zero, const Tv* p_, Tv* s, const Tv* q_, Tv* z,
                                                      const double* __restrict__ gpart, int ngp,
                                                      const double* __restrict__ dpart, int ndp,
                                                      double* __restrict__ gnew, int* __restrict__ flag) {
  using M = Mfma<Tv>;
  __shared__ Tv sl[128 * NR];
  __shared__ double red[256];
  __shared__ double gam[NR], del[NR];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, p = lane & 15, q = lane >> 4;
  Tv al = Tv(0);                       // of column tid % 16 = p
  if (p_) {
    colsum<256>(gpart, ngp, gam, red);
    colsum<256>(dpart, ndp, del, red);
    double alpha = 0.0;
    if (gam[p] != 0.0) {
      if (del[p] > 0.0) alpha = gam[p] / del[p];
      else if (blockIdx.x == 0 && tid < NR) atomicOr(flag, 1);
    }
    al = Tv(alpha);
  }
  double dacc = 0.0;
  for (int b = blockIdx.x; b < nblocks; b += gridDim.x) {
    const int s0 = off ? off[b] : b * stride;
    const int n = off ? off[b + 1] - s0 : stride;
    const int64_t o = int64_t(s0) * NR;
    __syncthreads();
    for (int i = tid; i < n * NR; i += 256) {
      Tv sn;
      if (p_) {
        e[o + i] = e_zero ? al * p_[o + i] : e[o + i] + al * p_[o + i];
        sn = s[o + i] - al * q_[o + i];
      } else {
        sn = src[o + i];
      }
      s[o + i] = sn;
      sl[i] = sn;
    }
    __syncthreads();
    const Tv* Mb = Minv + int64_t(b) * ld * ld;
    for (int sb = w; 16 * sb < n; sb += 4) {
      const int i = 16 * sb + p;
      typename M::acc_t acc = typename M::acc_t{Tv(0), Tv(0), Tv(0), Tv(0)};
      for (int k0 = 0; k0 < n; k0 += 32) {
        Tv a[8];
#pragma unroll
        for (int kb = 0; kb < 8; ++kb) {
          const int k = k0 + 4 * kb + q;
          a[kb] = k < n && i < n ? Mb[int64_t(k) * ld + i] : Tv(0);   // symmetric
        }
#pragma unroll
        for (int kb = 0; kb < 8; ++kb) {
          const int k = k0 + 4 * kb + q;
          if (k0 + 4 * kb < n) acc = M::mma(a[kb], k < n ? sl[k * NR + p] : Tv(0), acc);
        }
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int row = 16 * sb + M::row(t, q);
        if (row < n) {
          z[o + row * NR + p] = acc[t];
          dacc += double(sl[row * NR + p]) * double(acc[t]);
        }
      }
    }
  }
  colpart<256>(dacc, red, gnew);
}

// ------------------------------------------------------------ leaf bases
// xhat[leaf] (r x 16) = Q_leaf^T x_leaf: wave w takes slab w % ns of the rank
// and every (8 / ns)-th run of 16 points (ns = 1, 2, 4 slabs), the runs' sums
// meet in LDS.
template <typename Tq, typename Tv>
__global__ __launch_bounds__(512) void k_leaf_up16(const int* __restrict__ leaf_off, const Tq* __restrict__ Qr, int r,
                                                   const Tv* __restrict__ x, Tv* __restrict__ xhat) {
  using M = Mfma<Tv>;
  __shared__ Tv red[8][16 * NR];
  const int leaf = blockIdx.x;
  const int s0 = leaf_off[leaf], n = leaf_off[leaf + 1] - s0;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, p = lane & 15, q = lane >> 4;
  const int ns = r <= 16 ? 1 : r <= 32 ? 2 : 4, ng = 8 / ns;
  const int sb = w % ns, g = w / ns, j = 16 * sb + p;
  typename M::acc_t acc = typename M::acc_t{Tv(0), Tv(0), Tv(0), Tv(0)};
  for (int i0 = 16 * g; i0 < n; i0 += 16 * ng) {
    Tv a[4], b[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int i = i0 + 4 * t + q;
      a[t] = i < n && j < r ? ld_as<Tv, Tq>(Qr[int64_t(s0 + i) * r + j]) : Tv(0);
      b[t] = i < n ? x[int64_t(s0 + i) * NR + p] : Tv(0);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) acc = M::mma(a[t], b[t], acc);
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) red[w][M::row(t, q) * NR + p] = acc[t];
  __syncthreads();
  for (int e = threadIdx.x; e < r * NR; e += 512) {
    const int slab = e / (16 * NR), o = e % (16 * NR);
    Tv v = red[slab][o];
    for (int k = 1; k < ng; ++k) v += red[slab + k * ns][o];
    xhat[int64_t(leaf) * r * NR + e] = v;
  }
}

// out = alpha * (Q_leaf yhat_leaf + near) + beta * add, 64 rows of one leaf
// per workgroup, a slab of 16 rows per wave (tree order); yhat or near may be
// null, add is read only when beta != 0 (it may alias out).
template <typename Tq, typename Tv>
__global__ __launch_bounds__(256) void k_leaf_down16(const int* __restrict__ leaf_off, const Tq* __restrict__ Qc,
                                                     int r, const Tv* __restrict__ yhat,
                                                     const Tv* __restrict__ near_y,
                                                     const int* __restrict__ chunk_base, Tv* out, double alpha,
                                                     const Tv* add, double beta) {
  using M = Mfma<Tv>;
  const int leaf = blockIdx.x;
  const int s0 = leaf_off[leaf], n = leaf_off[leaf + 1] - s0;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, p = lane & 15, q = lane >> 4;
  const int r0 = 64 * int(blockIdx.y) + 16 * w, i = r0 + p;
  if (r0 >= n) return;
  typename M::acc_t acc = typename M::acc_t{Tv(0), Tv(0), Tv(0), Tv(0)};
  if (yhat) {
    const Tq* Q = Qc + int64_t(s0) * r + i;
    const Tv* yh = yhat + int64_t(leaf) * r * NR;
    for (int k0 = 0; k0 < r; k0 += 32) {
      Tv a[8], b[8];
#pragma unroll
      for (int kb = 0; kb < 8; ++kb) {
        const int k = k0 + 4 * kb + q;
        a[kb] = k < r && i < n ? ld_as<Tv, Tq>(Q[int64_t(k) * n]) : Tv(0);
        b[kb] = k < r ? yh[k * NR + p] : Tv(0);
      }
#pragma unroll
      for (int kb = 0; kb < 8; ++kb)
        if (k0 + 4 * kb < r) acc = M::mma(a[kb], b[kb], acc);
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int row = r0 + M::row(t, q);
    if (row >= n) continue;
    Tv v = acc[t];
    if (near_y) v += near_y[chunk_pos(chunk_base[leaf], chunk_len(n), row) * NR + p];
    const int64_t idx = int64_t(s0 + row) * NR + p;
    Tv o = Tv(alpha) * v;
    if (beta != 0.0) o += Tv(beta) * add[idx];
    out[idx] = o;
  }
}

// ------------------------------------------------------------ dispatch helpers
template <typename F>
void dispatch_T16(int T, F&& f) {
  switch (T) {
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    default: throw std::runtime_error("blocks of vectors need a rank of 9 to 64");
  }
}

// f(Tv{}, Te{}) for an operator precision p (vectors FP64 for P64, else FP32).
template <typename F>
void dispatch_prec(int p, F&& f) {
  if (p == P64) f(double{}, double{});
  else if (p == P32) f(float{}, float{});
  else f(float{}, bf16{});
}

// Levels per launch: n levels in equal shares, the coefficients of the lowest
// one at most 38 KB (with the level above half of it again, and the column
// sums, less than the 64 KB that a launch may use by default).
constexpr size_t SWEEP_LDS = 38912;
int levels_of(int n, int r, size_t vb) {
  int k = 1;
  while (k < 5 && (size_t(r) * NR * vb << (k + 1)) <= SWEEP_LDS) ++k;
  const int launches = (n + k - 1) / k;
  return (n + launches - 1) / launches;
}

}  // namespace

namespace {

// One launch each: the subtrees of nlev levels below depth q.
void sweep_up_launch(H2& h, int p, int q, int nlev, void* xall, const void* src, const void* prev, void* keep,
                     void* xroot, const double* gold, const double* gnew, int np) {
  const size_t lds = (size_t(h.r) * NR * (p == P64 ? 8 : 4) << nlev) * 3 / 2;
  dispatch_T16(h.T, [&](auto Tc) {
    constexpr int T = decltype(Tc)::value;
    dispatch_prec(p, [&](auto tv, auto te) {
      using Tv = decltype(tv);
      using Te = decltype(te);
      hipLaunchKernelGGL((k_sweep_up16<T, Te, Tv>), dim3(1u << q), dim3(SWEEP_NT), lds, h.stream, q, nlev, h.r,
                         static_cast<const Te*>(h.prec[p].E), static_cast<Tv*>(xall), static_cast<const Tv*>(src),
                         static_cast<const Tv*>(prev), static_cast<Tv*>(keep), static_cast<Tv*>(xroot), gold, gnew, np);
    });
  });
  check_launch("sweep_up16");
}

void sweep_down_launch(H2& h, int p, int q, int nlev, const void* yall, const void* root, const void* ybot, void* out,
                       const void* add, const void* xd, double* dpart) {
  const size_t lds = size_t(h.r) * NR * (p == P64 ? 8 : 4) << nlev;
  dispatch_T16(h.T, [&](auto Tc) {
    constexpr int T = decltype(Tc)::value;
    dispatch_prec(p, [&](auto tv, auto te) {
      using Tv = decltype(tv);
      using Te = decltype(te);
      hipLaunchKernelGGL((k_sweep_down16<T, Te, Tv>), dim3(1u << q), dim3(SWEEP_NT), lds, h.stream, q, nlev, h.r,
                         static_cast<const Te*>(h.prec[p].E), static_cast<const Tv*>(yall),
                         static_cast<const Tv*>(root), static_cast<const Tv*>(ybot), static_cast<Tv*>(out),
                         static_cast<const Tv*>(add), static_cast<const Tv*>(xd), dpart);
    });
  });
  check_launch("sweep_down16");
}

}  // namespace

void launch_sweep_up16(H2& h, int p, int d, void* xall, const void* src, const void* prev, const double* gold,
                       const double* gnew, int np) {
  const size_t vb = p == P64 ? 8 : 4;
  auto at = [&](int depth) { return static_cast<char*>(xall) + ((size_t(1) << depth) - 1) * h.r * NR * vb; };
  const int share = levels_of(std::max(d - h.d_top, 1), h.r, vb);
  bool first = true;
  for (int top = d; top > h.d_top || (first && src);) {
    const int nlev = std::min(share, top - h.d_top), q = top - nlev;
    sweep_up_launch(h, p, q, nlev, xall, first ? src : nullptr, first ? prev : nullptr,
                    first && src ? at(d) : nullptr, at(q), gold, gnew, np);
    top = q;
    first = false;
  }
}

int launch_sweep_down16(H2& h, int p, int d, void* yall, void* out, const void* add, const void* xd, double* dpart) {
  const size_t vb = p == P64 ? 8 : 4;
  auto at = [&](int depth) { return static_cast<char*>(yall) + ((size_t(1) << depth) - 1) * h.r * NR * vb; };
  const int share = levels_of(std::max(d - h.d_top, 1), h.r, vb);
  int blocks = 0;
  for (int q = h.d_top; q < d;) {
    const int nlev = (d - q) % share == 0 ? share : (d - q) % share;
    const bool last = q + nlev == d;
    sweep_down_launch(h, p, q, nlev, yall, at(q), at(q + nlev), last ? out : at(q + nlev), last ? add : nullptr, xd,
                      last ? dpart : nullptr);
    blocks = 1 << q;
    q += nlev;
  }
  return blocks;
}

void launch_restrict16(H2& h, int p, int k, const void* x, void* xnext) {
  if (k == 1) launch_leaf_up16(h, p, x, xnext);
  else sweep_up_launch(h, p, h.level_depth(k) - 1, 1, nullptr, x, nullptr, nullptr, xnext,
                       nullptr, nullptr, 0);
}

void launch_prolong16(H2& h, int p, int k, const void* enext, void* e) {
  if (k == 1) launch_leaf_down16(h, p, enext, nullptr, e, 1.0, e, 1.0);
  else sweep_down_launch(h, p, h.level_depth(k) - 1, 1, nullptr, enext, e, e, nullptr, nullptr, nullptr);
}

int launch_cg_step16_bj(H2& h, int p, int k, const void* src, void* e, bool e_zero, const void* pv, void* s,
                        const void* q, void* z, const double* gpart, int ngp, const double* dpart, int ndp,
                        double* gnew) {
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
    hipLaunchKernelGGL((k_cg_step16_bj<Tv>), dim3(grid), dim3(256), 0, h.stream, nb, off, h.r, M, ld,
                       static_cast<const Tv*>(src), static_cast<Tv*>(e), e_zero, static_cast<const Tv*>(pv),
                       static_cast<Tv*>(s), static_cast<const Tv*>(q), static_cast<Tv*>(z), gpart, ngp, dpart, ndp,
                       gnew, h.flags);
  });
  check_launch("cg_step16_bj");
  return grid;
}

void launch_leaf_up16(H2& h, int p, const void* x, void* xhat) {
  dispatch_prec(p, [&](auto tv, auto te) {
    using Tv = decltype(tv);
    using Te = decltype(te);
    hipLaunchKernelGGL((k_leaf_up16<Te, Tv>), dim3(h.nleaf), dim3(512), 0, h.stream, h.leaf_off,
                       static_cast<const Te*>(h.prec[p].Qr), h.r, static_cast<const Tv*>(x),
                       static_cast<Tv*>(xhat));
  });
  check_launch("leaf_up16");
}

void launch_leaf_down16(H2& h, int p, const void* yhat, const void* near_y, void* out, double alpha,
                        const void* add, double beta) {
  dispatch_prec(p, [&](auto tv, auto te) {
    using Tv = decltype(tv);
    using Te = decltype(te);
    hipLaunchKernelGGL((k_leaf_down16<Te, Tv>), dim3(h.nleaf, (h.leaf_max + 63) / 64), dim3(256), 0, h.stream,
                       h.leaf_off, static_cast<const Te*>(h.prec[p].Qc), h.r, static_cast<const Tv*>(yhat),
                       static_cast<const Tv*>(near_y), h.snear.chunk_base, static_cast<Tv*>(out), alpha,
                       static_cast<const Tv*>(add), beta);
  });
  check_launch("leaf_down16");
}

}  // namespace h2mg
