// Products with the H2 matrix (Section 3.1, matvec recursion after eq. h2)
// and with the restricted operators (Section 3.3, eq. a2_str), and the level
// transfers of Algorithm 1.
#include <hip/hip_runtime.h>

#include <stdexcept>
#include <string>
#include <vector>

#include "h2_build.h"

namespace h2mg {

namespace {

inline size_t vbytes(int p) { return p == P64 ? 8 : 4; }

// Pointer to the coefficients of depth d inside a gid-indexed buffer.
inline void* at_depth(void* base, int p, int d, int r) {
  return static_cast<char*>(base) + size_t((1 << d) - 1) * r * vbytes(p);
}
inline const void* at_depth(const void* base, int p, int d, int r) {
  return static_cast<const char*>(base) + size_t((1 << d) - 1) * r * vbytes(p);
}

// Everything of a fine product behind the leaf upsweep (x_L in xall).
void fine_from_leaves(H2& h, int p, const void* xt, void* out, bool to_user, double alpha, const void* add,
                      double beta) {
  void* xall = h.xall;
  void* yall = h.yall;
  const int r = h.r;
  bool near_done = false;
  if (h.d_top >= 0) {
    // upsweep: x_d = E^T x_{d+1}
    if (h.L > h.d_top) launch_sweep_up(h, p, h.L, xall, nullptr, nullptr, nullptr, nullptr, 0);
    // couplings of every depth in one launch, then one reduce for all depths
    near_done = p == P64 && !near_stored_for(h, p) && launch_near_far(h, xt, h.fine_launch, xall);
    if (!near_done) launch_gemv(h, p, h.fine_launch, xall);
    std::vector<const View*> vs;
    std::vector<int> bs;
    for (int d = h.d_top; d <= h.L; ++d) {
      vs.push_back(&h.sview[d]);
      bs.push_back(h.fine_launch.base[d - h.d_top]);
    }
    launch_reduce(h, p, h.d_top, h.L, vs.data(), bs.data(), nullptr, nullptr, yall, nullptr);
    // downsweep: y_d += E y_{d-1}
    launch_sweep_down(h, p, h.L, yall, at_depth(yall, p, h.L, r), nullptr, nullptr, nullptr);
  }
  // near field and leaf downsweep: y = D x + Q y_L
  if (near_stored_for(h, p)) launch_near_stored(h, p, xt);
  else if (!near_done) launch_near(h, p, xt);
  launch_fine_reduce(h, p, at_depth(yall, p, h.L, r), out, to_user, alpha, add, beta, xt);
}

}  // namespace

void apply_fine(H2& h, int p, const void* xt, void* out, double alpha, const void* add, double beta) {
  if (h.d_top >= 0) launch_leaf_up(h, p, xt, at_depth(h.xall, p, h.L, h.r));
  fine_from_leaves(h, p, xt, out, false, alpha, add, beta);
}

void apply_fine_user(H2& h, const double* x, double* y) {
  if (h.d_top >= 0)
    launch_leaf_up_gather(h, x, h.vtree, static_cast<double*>(at_depth(h.xall, P64, h.L, h.r)));
  else
    launch_gather(h, x, h.vtree);
  fine_from_leaves(h, P64, h.vtree, y, true, 1.0, nullptr, 0.0);
}

void* level_input(H2& h, int p, int k) { return at_depth(h.xall, p, h.level_depth(k), h.r); }

int apply_coarse(H2& h, int p, int k, const CoarseInput& in, void* y, const void* add, double* dpart) {
  const int d = h.level_depth(k);
  const int r = h.r;
  void* xall = h.xall;
  void* yall = h.yall;
  launch_sweep_up(h, p, d, xall, in.src, in.prev, in.gold, in.gnew, in.np);
  const Launch& l = h.coarse_launch[d];
  launch_gemv(h, p, l, xall);
  // partial sums of every depth: S_q for q < d, Pi_d and S_d at depth d
  std::vector<const View*> v0, v1;
  std::vector<int> b0, b1;
  for (int q = h.d_top; q < d; ++q) {
    v0.push_back(&h.sview[q]);
    b0.push_back(l.base[q - h.d_top]);
    v1.push_back(nullptr);
    b1.push_back(0);
  }
  const int nv = d - h.d_top;
  v0.push_back(&h.pview[d]);
  b0.push_back(l.base[nv]);
  v1.push_back(&h.sview[d]);
  b1.push_back(l.base[nv + 1]);
  launch_reduce(h, p, h.d_top, d, v0.data(), b0.data(), v1.data(), b1.data(), yall,
                d == h.d_top ? y : nullptr);
  // downsweep, the last step writing the output
  if (d > h.d_top) return launch_sweep_down(h, p, d, yall, y, add, at_depth(xall, p, d, r), dpart);
  const int64_t n = int64_t(1 << d) * r;
  const int vp = p == P64 ? P64 : P32;
  if (add) launch_axpby(h, vp, n, 1.0, add, -1.0, y);
  if (!dpart) return 0;
  launch_dot(h, vp, n, at_depth(xall, p, d, r), y, dpart);
  return dot_parts(n);
}

void apply_coarse(H2& h, int p, int k, const void* x, void* y) {
  apply_coarse(h, p, k, CoarseInput{x}, y, nullptr, nullptr);
}

void residual_level(H2& h, int p, int k, const void* x, void* out, const void* b) {
  if (k == 1) apply_fine(h, p, x, out, -1.0, b, 1.0);
  else apply_coarse(h, p, k, CoarseInput{x}, out, b, nullptr);
}

void restrict_level(H2& h, int p, int k, const void* r, void* r_next) {
  if (k == 1) launch_leaf_up(h, p, r, r_next);
  else launch_transfer_up(h, p, h.level_depth(k) - 1, r, r_next);
}

void prolong_level(H2& h, int p, int k, const void* e_next, void* e, const void* add, double beta) {
  if (k == 1) launch_leaf_down(h, p, e_next, e, 1.0, add, beta);
  else {
    if (add && beta != 1.0) throw std::runtime_error("prolongation supports beta = 1 only");
    launch_transfer_down(h, p, h.level_depth(k) - 1, e_next, e, add);
  }
}

}  // namespace h2mg
