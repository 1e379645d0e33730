// Device-side helpers shared by the setup and apply kernels.
//
// Tiled block layout.  Every r x r block (couplings S, projected close
// blocks, transfers E) is stored for a 64-lane wave laid out as an 8 x 8
// lane grid: lane l = 8a + b owns rows a*T .. a*T+T-1 and columns
// b*T .. b*T+T-1 of the block, where T is the smallest power of two with
// 8T >= r (entries beyond r are zero).  The T*T elements of a lane are cut
// into chunks of K consecutive elements (K = min(16 bytes / element size,
// T*T)).  Only the A x A lanes with rows and columns below r take part, A =
// ceil(r / T): chunk c of lane (a, b) lives at element offset
// (c*A*A + a*A + b)*K, so a wave reads each chunk row as one contiguous
// segment of A*A*K elements and the used part of a tile is contiguous too.
// A tile takes tile_elems(T) elements whatever A is.  With all 64 lanes'
// places stored, a block of rank 27 streamed 1024 entries for 729 (now 784),
// and a 49-point near-field tile 4096 for 2401 (now 3136).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <limits>
#include <type_traits>

namespace h2mg {

// ---------------------------------------------------------------- bf16
struct bf16 {
  uint16_t bits;
};

__host__ __device__ inline float bf16_to_float(bf16 v) {
  union { uint32_t u; float f; } c;
  c.u = uint32_t(v.bits) << 16;
  return c.f;
}

// Round-to-nearest-even of an FP32 value to BF16 (finite inputs).
__host__ __device__ inline bf16 float_to_bf16(float f) {
  union { uint32_t u; float f; } c;
  c.f = f;
  uint32_t lsb = (c.u >> 16) & 1u;
  bf16 r;
  r.bits = uint16_t((c.u + 0x7fffu + lsb) >> 16);
  return r;
}

template <typename T> struct Conv;
template <> struct Conv<double> {
  __device__ static double to_f64(double v) { return v; }
  __device__ static double from_f64(double v) { return v; }
};
template <> struct Conv<float> {
  __device__ static double to_f64(float v) { return v; }
  __device__ static float from_f64(double v) { return float(v); }
};
template <> struct Conv<bf16> {
  __device__ static double to_f64(bf16 v) { return bf16_to_float(v); }
  __device__ static bf16 from_f64(double v) { return float_to_bf16(float(v)); }
};

// Load one stored element as the accumulation type.
template <typename Tacc, typename Tb> __device__ inline Tacc ld_as(Tb v);
template <> __device__ inline double ld_as<double, double>(double v) { return v; }
template <> __device__ inline float ld_as<float, float>(float v) { return v; }
template <> __device__ inline float ld_as<float, bf16>(bf16 v) { return bf16_to_float(v); }
template <> __device__ inline double ld_as<double, float>(float v) { return v; }

// ---------------------------------------------------------------- tiles
__host__ __device__ constexpr int tile_T(int r) {
  return r <= 8 ? 1 : r <= 16 ? 2 : r <= 32 ? 4 : 8;
}
template <typename Tb>
__host__ __device__ constexpr int tile_K(int T) {
  return (16 / int(sizeof(Tb))) < T * T ? (16 / int(sizeof(Tb))) : T * T;
}
// Lanes per side that hold entries of a block of r rows.
__host__ __device__ constexpr int tile_A(int r, int T) { return (r + T - 1) / T; }
// Elements per stored tile.
__host__ __device__ constexpr int64_t tile_elems(int T) { return 64LL * T * T; }

// Element offset of block entry (i, j) inside a tile (i, j < A * T).
template <typename Tb>
__host__ __device__ inline int tile_offset(int i, int j, int T, int A) {
  const int K = tile_K<Tb>(T);
  const int a = i / T, u = i % T, b = j / T, v = j % T;
  const int e = u * T + v;
  return ((e / K) * A * A + A * a + b) * K + (e % K);
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Load the T*T elements of this lane's sub-tile (row-major u*T + v) from
// the tile starting at `tile`.  Lanes that hold no entries get those of
// another one: their rows and columns meet zero coefficients, and their own
// results are not used.  NT: non-temporal (streaming) loads, for
// blocks read once per product so they do not evict reused vectors.  PARTS:
// only rows [part T / PARTS, (part + 1) T / PARTS) of the sub-tile.
template <int T, typename Tb, typename Tacc, bool NT = false, int PARTS = 1>
__device__ inline void load_subtile(const Tb* __restrict__ tile, int lane, int A, Tacc (&B)[T * T / PARTS],
                                    int part = 0) {
  constexpr int K = tile_K<Tb>(T);
  constexpr int NC = T * T / K / PARTS;
  static_assert(NC * K * PARTS == T * T);
  tile += part * NC * A * A * K;
  // a uniform base and one 32-bit lane offset for all chunks (an address per
  // chunk would take 64 registers)
  const uint32_t off = uint32_t(A * min(lane >> 3, A - 1) + min(lane & 7, A - 1)) * uint32_t(K * sizeof(Tb));
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const Tb* p = reinterpret_cast<const Tb*>(reinterpret_cast<const char*>(tile + c * A * A * K) + off);
    if constexpr (K * sizeof(Tb) == 16) {
      // one 16-byte load per chunk
      union { u32x4 q; Tb e[K]; } u;
      if constexpr (NT) u.q = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
      else u.q = *reinterpret_cast<const u32x4*>(p);
#pragma unroll
      for (int k = 0; k < K; ++k) B[c * K + k] = ld_as<Tacc, Tb>(u.e[k]);
    } else {
#pragma unroll
      for (int k = 0; k < K; ++k) B[c * K + k] = ld_as<Tacc, Tb>(p[k]);
    }
  }
}

// ---------------------------------------------------------------- near-field chunks
// Position of point i of a leaf of n points in the chunk-padded order of the
// stored near field: ceil(n / 64) chunks of equal length (the last one
// shorter), each padded to 64, the first one at chunk `base`.
__host__ __device__ inline int chunk_len(int n) {
  const int k = (n + 63) / 64;
  return (n + k - 1) / k;
}
__device__ inline int64_t chunk_pos(int base, int len, int i) {
  const int c = (i >= len) + (i >= 2 * len) + (i >= 3 * len);   // at most 256 points
  return int64_t(base + c) * 64 + (i - c * len);
}

// ---------------------------------------------------------------- matrix cores
// 16 x 16 x 4 products: lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16]; accumulator element t of lane l is row row(t, l / 16),
// column l % 16 (measured on gfx950).
typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
template <typename Tc> struct Mfma;
template <> struct Mfma<double> {
  typedef d4 acc_t;
  __device__ static d4 mma(double a, double b, d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  __device__ static int row(int t, int q) { return 4 * t + q; }
};
template <> struct Mfma<float> {
  typedef f4 acc_t;
  __device__ static f4 mma(float a, float b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  __device__ static int row(int t, int q) { return 4 * q + t; }
};

// ---------------------------------------------------------------- kernels
enum { KER_EXP = 0, KER_GAUSS = 1, KER_MATERN32 = 2, KER_LAPLACE = 3 };
// deriv: the kernel itself, its derivative in the length scale at fixed r,
// or g(r) = k'(r) / r (0 at r = 0, where its self term cancels in the
// coordinate gradient).
enum { DER_NONE = 0, DER_LENGTH = 1, DER_RADIAL = 2 };

struct KernelParams {
  int kind;
  int deriv;
  double inv_l;        // 1 / l
  // k = f(z) 2^(c s) with s = r, or r^2 for the Gaussian: the constants of both,
  // each rounded once from extended precision
  double c;            // -log2(e) / l; Gaussian -log2(e) / (2 l^2); Matern -sqrt(3) log2(e) / l
  double z;            // z / s: 1 / l; Matern sqrt(3) / l
  double far;          // the s from which on 2^(c s) is 0 in FP64: 1100 / -c
  double shift;
};
// What a kernel evaluation needs of them, in its precision.
template <typename T>
struct KernelConst {
  T inv_l, c, z, far;
  __host__ __device__ explicit KernelConst(const KernelParams& kp)
      : inv_l(T(kp.inv_l)), c(T(kp.c)), z(T(kp.z)), far(T(kp.far)) {}
};

// Square root, reciprocal square root and exponential of the kernels.  The
// products that evaluate their close blocks spend nearly all their time here
// (FP64 vector issue), and the arguments are known: x = r^2 >= 0 and an
// exponent <= 0.  So nothing is spent on signs, special cases and subnormal
// scaling: a Matern entry with its distance and its two sums issues 32
// operations, most of them FP64, instead of 66 with the library's sqrt and exp
// (a product at N = 131072, 3D, close blocks evaluated: 3453 to 2398 us).
//   sqrt_nn: from the hardware's reciprocal square root y (about 2^-24 off in
//     FP64, 1 ulp in FP32), g = x y and the exact residual d = x - g^2 =
//     e g^2: sqrt(x) = g + d y (1/2 + 3/8 e) + O(e^3), within 0.501 ulp.
//     At x = 0 only the reciprocal root is kept finite, and the root is 0.  (The
//     hardware's FP64 reciprocal root takes subnormals, measured; its FP32 one
//     does not.)  MINED arguments start at MIN_R2, whose root is too small to
//     matter.
//   rsqrt_nn: Newton's iteration.
//   exp2_prod(s, c) = 2^(c s), c s <= 0: n = rint(c s), f = c s - n with one
//     rounding (the product's own rounding, up to |c s| times larger, does not
//     occur), 2^f = 1 + f q(f) with q the degree-10 interpolant of (2^f - 1) / f
//     in the Chebyshev nodes of [-1/2, 1/2] (2e-17 off), scaled by 2^n exactly;
//     2^0 is exactly 1.  s is lowered to where 2^(c s) is 0 (an overflowed r^2,
//     whose root is a NaN here, ends up there too).  In FP32 the hardware's 2^w
//     (1 ulp) of the rounded product; it flushes subnormal results, which are
//     scaled into its range unless there are none (NORMAL).
template <typename T> constexpr T MIN_R2 = T(0);
template <> inline constexpr double MIN_R2<double> = 1e-290;
template <> inline constexpr float MIN_R2<float> = 1e-36f;

template <bool MINED = false>
__device__ inline double sqrt_nn(double x) {
  const double y = __builtin_amdgcn_rsq(MINED ? x : __builtin_fmax(x, 0x1p-1074));
  const double g = x * y;
  const double t = __builtin_fma(-g, g, x) * y;
  return __builtin_fma(t, __builtin_fma(0.375, t * y, 0.5), g);
}
template <bool MINED = false>
__device__ inline float sqrt_nn(float x) {
  const bool small = !MINED && x < 1e-28f;       // the residual below would be subnormal
  if constexpr (!MINED) x = small ? x * 0x1p64f : x;
  const float y = __builtin_amdgcn_rsqf(MINED ? x : __builtin_fmaxf(x, MIN_R2<float>));
  const float g = x * y;
  const float s = __builtin_fmaf(__builtin_fmaf(-g, g, x), 0.5f * y, g);
  return small ? s * 0x1p-32f : s;
}
__device__ inline double rsqrt_nn(double x) {
  double y = __builtin_amdgcn_rsq(x);
  double e = __builtin_fma(-x * y, y, 1.0);
  y = __builtin_fma(y * e, __builtin_fma(0.375, e, 0.5), y);
  e = __builtin_fma(-x * y, y, 1.0);
  return __builtin_fma(0.5 * y, e, y);
}
__device__ inline float rsqrt_nn(float x) {
  const bool small = x < 1.1754944e-38f;         // the hardware's root takes no subnormals
  x = small ? x * 0x1p64f : x;
  const float y = __builtin_amdgcn_rsqf(x);
  const float s = __builtin_fmaf(0.5f * y, __builtin_fmaf(-x * y, y, 1.0f), y);
  return small ? s * 0x1p32f : s;
}
template <bool NORMAL = false>
__device__ inline double exp2_prod(double s, double c) {
  constexpr double MAGIC = 6755399441055744.0;   // 1.5 * 2^52: w + MAGIC holds rint(w) in its low bits
  const double t = __builtin_fma(s, c, MAGIC);
  const double f = __builtin_fma(s, c, -(t - MAGIC));
  double q = 4.4549605981865186e-10;
  q = __builtin_fma(q, f, 7.072585949269223e-09);
  q = __builtin_fma(q, f, 1.0178062445845774e-07);
  q = __builtin_fma(q, f, 1.321544258792169e-06);
  q = __builtin_fma(q, f, 1.525273382983612e-05);
  q = __builtin_fma(q, f, 0.0001540353044173605);
  q = __builtin_fma(q, f, 0.0013333558146416936);
  q = __builtin_fma(q, f, 0.009618129107606888);
  q = __builtin_fma(q, f, 0.0555041086648216);
  q = __builtin_fma(q, f, 0.24022650695910097);
  q = __builtin_fma(q, f, 0.6931471805599453);
  return __builtin_ldexp(__builtin_fma(q, f, 1.0), int(__double2loint(t)));
}
template <bool NORMAL = false>
__device__ inline float exp2_prod(float s, float c) {
  const float w = s * c;
  if constexpr (NORMAL) return __builtin_amdgcn_exp2f(w);
  const bool small = w < -126.0f;
  return __builtin_amdgcn_exp2f(small ? w + 64.0f : w) * (small ? 0x1p-64f : 1.0f);
}
__device__ inline double lower_to(double s, double hi) { return __builtin_fmin(s, hi); }
__device__ inline float lower_to(float s, float hi) { return __builtin_fminf(s, hi); }

// k (or its derivative) as a function of the squared distance (no shift),
// for a kernel fixed at compile time.  MINED: r2 is finite and at least MIN_R2
// (r = 0 included, so not for the kernels that ask for r2 = 0), and the exponent
// above -2^30: nothing is lowered.  NORMAL: the exponent is above -126 (FP32).
template <int KIND, int DERIV, typename T, bool MINED = false, bool NORMAL = false>
__device__ inline T kernel_fixed(const KernelConst<T>& k, T r2) {
  auto lower = [&](T s) { return MINED ? s : lower_to(s, k.far); };
  if constexpr (KIND == KER_LAPLACE) {
    // 1 / (4 pi r); 0 at r = 0 (the matrix supplies its own diagonal) and for an
    // overflowed r^2
    return r2 == T(0) || r2 > std::numeric_limits<T>::max() ? T(0) : T(0.07957747154594767) * rsqrt_nn(r2);
  }
  if constexpr (DERIV == DER_RADIAL) {
    if (r2 == T(0)) return T(0);
  }
  if constexpr (KIND == KER_GAUSS) {
    const T s = lower(r2);
    const T e = exp2_prod<NORMAL>(s, k.c);
    if constexpr (DERIV == DER_NONE) return e;
    else if constexpr (DERIV == DER_LENGTH) return s * (k.inv_l * k.inv_l) * (k.inv_l * e);   // 1 / l^3 may overflow
    else return -k.inv_l * k.inv_l * e;
  } else if constexpr (KIND == KER_EXP) {
    const T rr = lower(sqrt_nn<MINED>(r2));
    const T e = exp2_prod<NORMAL>(rr, k.c);
    if constexpr (DERIV == DER_NONE) return e;
    else if constexpr (DERIV == DER_LENGTH) return rr * (k.inv_l * k.inv_l) * e;
    else return -k.inv_l * e / rr;
  } else {
    const T rr = lower(sqrt_nn<MINED>(r2));
    const T e = exp2_prod<NORMAL>(rr, k.c);
    if constexpr (DERIV == DER_NONE) return (T(1) + rr * k.z) * e;
    else if constexpr (DERIV == DER_LENGTH) return (rr * k.z) * (rr * k.z) * k.inv_l * e;
    else return T(-3) * k.inv_l * k.inv_l * e;
  }
}

// Call f(integral_constant<KIND>, integral_constant<DERIV>) for a runtime pair.
template <typename F>
__host__ __device__ inline void dispatch_kernel(int kind, int deriv, F&& f) {
  using I = int;
  auto d = [&](auto kc) {
    if (deriv == DER_LENGTH) f(kc, std::integral_constant<I, DER_LENGTH>{});
    else if (deriv == DER_RADIAL) f(kc, std::integral_constant<I, DER_RADIAL>{});
    else f(kc, std::integral_constant<I, DER_NONE>{});
  };
  if (kind == KER_GAUSS) d(std::integral_constant<I, KER_GAUSS>{});
  else if (kind == KER_EXP) d(std::integral_constant<I, KER_EXP>{});
  else if (kind == KER_LAPLACE)   // no length scale, so no derivative kernels
    f(std::integral_constant<I, KER_LAPLACE>{}, std::integral_constant<I, DER_NONE>{});
  else d(std::integral_constant<I, KER_MATERN32>{});
}

__device__ inline double kernel_r2(const KernelParams& kp, double r2) {
  double v = 0.0;
  dispatch_kernel(kp.kind, kp.deriv, [&](auto kc, auto dc) {
    v = kernel_fixed<decltype(kc)::value, decltype(dc)::value, double>(KernelConst<double>(kp), r2);
  });
  return v;
}

// Per-point scale s (on rows and columns) and diagonal d of the scaled form
// diag(s) K diag(s) + diag(d), tree order; null pointers mean s = 1 and
// d = the constant shift.  Optional quadrature of the close entries: point i
// carries nq sub-points qy[i] (nq x dim, row-major) with weights qu[i] (nq),
// and the entry between distinct points i, j of a close leaf pair is
// sum_p sum_q qu[i][p] qu[j][q] k(|qy[i][p] - qy[j][q]|) (the weights carry
// any scaling; far blocks keep the point values).
struct PointScale {
  const double* s;
  const double* d;
  const double* qy;
  const double* qu;
  int nq;
};

// One entry of the scaled matrix from the kernel value k between tree
// positions i and j (self: the same point).
__device__ inline double scaled_entry(double k, int64_t i, int64_t j, bool self, const PointScale& ps,
                                      double shift) {
  if (ps.s) k *= ps.s[i] * ps.s[j];
  if (self) k += ps.d ? ps.d[i] : shift;
  return k;
}

// The close entry (i, j) of a leaf pair: the point kernel value (squared
// distance r2 of the two points) in the scaled form, or the quadrature sum
// when the close entries are given by quadrature (its diagonal is d or the
// shift).
__device__ inline double near_entry(const KernelParams& kp, const PointScale& ps, int dim, double r2,
                                    int64_t i, int64_t j, bool self) {
  if (!ps.qy) return scaled_entry(kernel_r2(kp, r2), i, j, self, ps, kp.shift);
  if (self) return ps.d ? ps.d[i] : kp.shift;
  const int nq = ps.nq;
  const double* yi = ps.qy + i * nq * dim;
  const double* yj = ps.qy + j * nq * dim;
  const double* ui = ps.qu + i * nq;
  const double* uj = ps.qu + j * nq;
  double sum = 0.0;
  for (int p = 0; p < nq; ++p) {
    double part = 0.0;
    for (int q = 0; q < nq; ++q) {
      double d2 = 0.0;
      for (int a = 0; a < dim; ++a) {
        const double dx = yi[p * dim + a] - yj[q * dim + a];
        d2 += dx * dx;
      }
      part += uj[q] * kernel_r2(kp, d2);
    }
    sum += ui[p] * part;
  }
  return sum;
}

// ---------------------------------------------------------------- shuffles
__device__ inline double shfl_xor(double v, int m) { return __shfl_xor(v, m, 64); }
__device__ inline float shfl_xor(float v, int m) { return __shfl_xor(v, m, 64); }

// Sum over the 8 lanes that share b (lane bits 3..5 = a) of T values each,
// as a butterfly transpose-reduce: afterwards lane (a, b) holds the full sum
// of value index a (T = 8), or of index a >> (3 - log2 T) for smaller T.
template <int T, typename Tv>
__device__ inline Tv transpose_reduce_a(Tv (&z)[T], int a) {
  if constexpr (T == 1) {
    Tv s = z[0];
    s += shfl_xor(s, 8);
    s += shfl_xor(s, 16);
    s += shfl_xor(s, 32);
    return s;
  } else {
    // halve the value set at each step, masks 32, 16, 8 (a bits 2, 1, 0)
    constexpr int H = T / 2;
    const bool hi = (a >> 2) & 1;
    Tv v1[H];
#pragma unroll
    for (int k = 0; k < H; ++k) {
      const Tv keep = hi ? z[k + H] : z[k];
      const Tv send = hi ? z[k] : z[k + H];
      v1[k] = keep + shfl_xor(send, 32);
    }
    if constexpr (H == 1) {
      Tv s = v1[0];
      s += shfl_xor(s, 16);
      s += shfl_xor(s, 8);
      return s;
    } else {
      constexpr int Q = H / 2;
      const bool mid = (a >> 1) & 1;
      Tv v2[Q];
#pragma unroll
      for (int k = 0; k < Q; ++k) {
        const Tv keep = mid ? v1[k + Q] : v1[k];
        const Tv send = mid ? v1[k] : v1[k + Q];
        v2[k] = keep + shfl_xor(send, 16);
      }
      if constexpr (Q == 1) {
        Tv s = v2[0];
        s += shfl_xor(s, 8);
        return s;
      } else {
        const bool lo = a & 1;
        const Tv keep = lo ? v2[1] : v2[0];
        const Tv send = lo ? v2[0] : v2[1];
        return keep + shfl_xor(send, 8);
      }
    }
  }
}

// Value index held by lane a after transpose_reduce_a.
template <int T>
__device__ inline int reduced_index(int a) {
  if constexpr (T == 1) return 0;
  else if constexpr (T == 2) return (a >> 2) & 1;
  else if constexpr (T == 4) return ((a >> 2) & 1) * 2 + ((a >> 1) & 1);
  else return ((a >> 2) & 1) * 4 + ((a >> 1) & 1) * 2 + (a & 1);
}

}  // namespace h2mg
