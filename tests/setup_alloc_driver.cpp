// Host driver of tests/test_host_setup_alloc.py: the hierarchy setup (csrc/h2_build.cpp) with the HIP
// runtime and the kernels replaced by host stand-ins, so that any one device allocation can be refused.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <random>
#include <vector>

#include "h2_build.h"

namespace {

int g_left = -1;                       // allocations that still succeed (-1: all)
bool g_not_spd = false;

}  // namespace

extern "C" {
hipError_t hipMalloc(void** p, size_t bytes) {
  if (g_left == 0) return hipErrorOutOfMemory;
  if (g_left > 0) --g_left;
  *p = std::calloc(1, bytes);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stand-in"; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t*) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float*, hipEvent_t, hipEvent_t) { return hipSuccess; }
}

namespace h2mg {

void launch_leaf_basis_qr(H2&) {}
void launch_transfer_qr(H2&, int) {}
void launch_couplings(H2&, int) {}
void launch_pi_leaf(H2&) {}
void launch_pi_upper(H2&, int, const int*) {}
void launch_assemble_dense(H2&, double*, int64_t) {}
void launch_assemble_kernel_dense(H2&, double*, int64_t) {}
void launch_potrf(H2& h, double*, int64_t, double*) { h.flags[0] = g_not_spd; }
void launch_tri_inverse(H2&, const double*, int64_t, double*, double*) {}
void launch_cast_precision(H2&, int) {}
void launch_near_tiles(H2&) {}
void launch_cast_near_tiles(H2&) {}
void launch_gather(H2&, const double*, double*) {}
void launch_gather_rows(H2&, int, const double*, double*) {}
void launch_scatter_rows(H2&, const double*, double*) {}
void launch_dot(H2&, int, int64_t, const void*, const void*, double*) {}
void launch_axpby(H2&, int, int64_t, double, const void*, double, void*) {}
void launch_coord_mul(H2&, int, const double*, double*) {}
void launch_coord_grad(H2&, int, double, const double*, const double*, const double*, double*) {}
void apply_fine(H2&, int, const void*, void*, double, const void*, double) {}
int dot_parts(int64_t) { return 1; }

}  // namespace h2mg

using namespace h2mg;

#define CHECK(c)                                                        \
  do {                                                                  \
    if (!(c)) {                                                         \
      std::printf("line %d: %s (%s)\n", __LINE__, #c, last_error_cstr()); \
      return 1;                                                         \
    }                                                                   \
  } while (0)

int main() {
  const int n = 600;
  std::mt19937_64 rng(7);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  std::vector<double> pts(2 * n);
  for (double& v : pts) v = u(rng);
  const h2mg_kernel kernel{KER_EXP, 0.1, 1.0, 0};
  for (double eta : {0.7, 1e-9}) {     // with far blocks and without
    const h2mg_build_opts opts{20, eta, 3};
    H2* h = nullptr;
    CHECK(build_h2(pts.data(), n, 2, &kernel, &opts, nullptr, &h) == H2MG_OK);
    CHECK((h->d_top >= 0) == (eta > 0.1));
    const size_t bytes = h->arena.bytes, count = h->arena.ptrs.size();
    auto untouched = [&] {
      return !h->mg_built && !h->chol && !h->cinv && !h->cdiag && h->arena.bytes == bytes && h->arena.ptrs.size() == count;
    };
    // an operator that is not positive definite, twice
    g_not_spd = true;
    for (int k = 0; k < 2; ++k) {
      CHECK(setup_mg(*h, 0) == H2MG_ERR_NOT_SPD);
      CHECK(untouched());
    }
    g_not_spd = false;
    // every allocation before that of the inverse refused in turn: out of memory, nothing kept
    int ok = 0;
    for (; ok < 100; ++ok) {
      g_left = ok;
      const h2mg_status st = setup_mg(*h, 0);
      g_left = -1;
      if (st == H2MG_OK) break;
      CHECK(st == H2MG_ERR_OOM);
      CHECK(untouched());
    }
    // the first attempt that succeeds lacks the inverse only
    const size_t square = size_t(h->Nl) * h->Nl * sizeof(double);
    CHECK(h->mg_built && h->chol && !h->cinv && !h->cdiag);
    CHECK(h->arena.bytes == bytes + square && h->arena.ptrs.size() == count + 1);
    delete h;
    // and with room for everything the inverse, which then holds the factor too
    CHECK(build_h2(pts.data(), n, 2, &kernel, &opts, nullptr, &h) == H2MG_OK);
    CHECK(setup_mg(*h, 0) == H2MG_OK && !h->chol && h->cinv && h->cdiag);
    CHECK(h->arena.bytes == bytes + square + size_t(h->Nl) * sizeof(double));
    delete h;
  }
  std::printf("all checks passed\n");
  return 0;
}
