// nlbm_fwd.hip -- instances and launch of the learned-collision step kernel
// (kernels_fwd.hpp), in a translation unit of its own: it is built with the
// max-ILP instruction scheduler, which the library's other kernels do not
// take (several of them need more registers with it).
#include <hip/hip_runtime.h>

#include "kernels_fwd.hpp"
#include "step_rule.hpp"

namespace lbm {

namespace {

// Launches the instance for work items of form M; with halves > 0 only where
// there are at most halves / 2 items per wavefront (else launched stays false).
template <class L, int H, int P, bool FORCED, int M>
hipError_t fwd_items(int ncu, hipStream_t s, const float* Ain, float* Aout, const float* theta,
                     Grid G, Force Fc, float rho0, float omega, float knn, int nitems, int nxc,
                     int halves, bool& launched) {
  const auto kernel = nlbm_step_kernel<L, H, P, FORCED, M>;
  constexpr int wb = StepLds<L, H, M>::waves_per_block(P, FORCED);
  int occ = 1;  // (FLAT16: no more than one workgroup per compute unit)
  if (M != FLAT16) {
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kernel, 64 * wb, 0);
    if (e != hipSuccess) return e;
  }
  launched = halves == 0 || 2LL * nitems <= (long long)halves * ncu * occ * wb;
  if (!launched) return hipSuccess;
  hipLaunchKernelGGL(kernel, dim3(persistent_grid(ncu, occ, wb, nitems)), dim3(64 * wb), 0, s,
                     Ain, Aout, theta, G, Fc, rho0, omega, knn, nitems, nxc,
                     StepDiv<M>::of(G));
  return hipGetLastError();
}

// The form of the work items.
//
// Small grids: 16 nodes per wavefront instead of 64, since most of a step's
// time is then one wavefront's chain: the staging of the weights, the loads,
// four dependent network evaluations one after the other, the stores.  In
// workgroups of four while one per compute unit holds all items, else of
// eight (fewer stage the weights).  us per step, 64 / 16 nodes: D2Q9 64^2 fp32
// H = 32 8.2 / 5.2, bf16 H = 64 13.2 / 6.7, 256^2 13.8 / 9.3; D3Q19 bf16 16^3
// 15.6 / 8.1, 32^3 16.1 / 8.9.  Up to one, one and a half or two items per
// wavefront: step_item_halves.
// All forms give the same bits: the collision's sums have their roundings
// written out (a network rounded to 16 bits makes 1e-5 of a last-bit
// difference within ten steps).
//
// Else 64 nodes: of one row, whose addresses are scalar but for the x part, or
// in flat order, where no lane is idle at the rows' ends and the addresses
// cost some 60 more instructions per item: D3Q19 fp16 150 x 131 x 117 (22% idle)
// 137 / 117 us, bf16 120 x 128 x 128 (6%) 88 / 85 us, D2Q9 1000^2 (2.3%) 38.4
// / 38.4 us, without idle lanes 88.2 / 90.1 us (128^3): flat from 3%.
template <class L, int H, int P, bool FORCED>
hipError_t fwd_one(int ncu, hipStream_t s, const float* Ain, float* Aout, const float* theta,
                   Grid G, Force Fc, float rho0, float omega, float knn) {
  const int nxc = (G.nx + 63) / 64;
  const long long nodes = (long long)G.plane * G.batch, rows = nodes / G.nx;
  const int n16 = (int)((nodes + 15) / 16), n64 = (int)((nodes + 63) / 64);
  bool launched;
  if (n16 <= 4 * ncu)
    return fwd_items<L, H, P, FORCED, FLAT16>(ncu, s, Ain, Aout, theta, G, Fc, rho0, omega, knn,
                                              n16, nxc, 0, launched);
  if (n16 <= 2 * 32 * ncu) {  // (a compute unit holds 32 wavefronts at most)
    constexpr int halves = step_item_halves(L::Q, H, P == P_F32, FORCED);
    hipError_t e = fwd_items<L, H, P, FORCED, FLAT16W>(ncu, s, Ain, Aout, theta, G, Fc, rho0,
                                                       omega, knn, n16, nxc, halves, launched);
    if (launched || e != hipSuccess) return e;
  }
  if (32LL * 64 * nxc >= 33LL * G.nx)
    return fwd_items<L, H, P, FORCED, FLAT64>(ncu, s, Ain, Aout, theta, G, Fc, rho0, omega, knn,
                                              n64, nxc, 0, launched);
  return fwd_items<L, H, P, FORCED, ROWS64>(ncu, s, Ain, Aout, theta, G, Fc, rho0, omega, knn,
                                            (int)(rows * nxc), nxc, 0, launched);
}

template <class L, int H, int P>
hipError_t fwd_forced(bool forced, int ncu, hipStream_t s, const float* Ain, float* Aout,
                      const float* theta, Grid G, Force Fc, float rho0, float omega, float knn) {
  // forced and unforced instances: the unforced one needs fewer registers
  if (forced)
    return fwd_one<L, H, P, true>(ncu, s, Ain, Aout, theta, G, Fc, rho0, omega, knn);
  return fwd_one<L, H, P, false>(ncu, s, Ain, Aout, theta, G, Fc, rho0, omega, knn);
}

template <class L, int H>
hipError_t fwd_prec(int prec, bool forced, int ncu, hipStream_t s, const float* Ain, float* Aout,
                    const float* theta, Grid G, Force Fc, float rho0, float omega, float knn) {
  switch (prec) {
    case P_F32:
      return fwd_forced<L, H, P_F32>(forced, ncu, s, Ain, Aout, theta, G, Fc, rho0, omega, knn);
    case P_BF16:
      return fwd_forced<L, H, P_BF16>(forced, ncu, s, Ain, Aout, theta, G, Fc, rho0, omega, knn);
    default:
      return fwd_forced<L, H, P_F16>(forced, ncu, s, Ain, Aout, theta, G, Fc, rho0, omega, knn);
  }
}

template <class L>
hipError_t fwd_hidden(int hidden, int prec, bool forced, int ncu, hipStream_t s,
                      const float* Ain, float* Aout, const float* theta, Grid G, Force Fc,
                      float rho0, float omega, float knn) {
  if (hidden == 32)
    return fwd_prec<L, 32>(prec, forced, ncu, s, Ain, Aout, theta, G, Fc, rho0, omega, knn);
  return fwd_prec<L, 64>(prec, forced, ncu, s, Ain, Aout, theta, G, Fc, rho0, omega, knn);
}

}  // namespace

hipError_t nlbm_fwd_launch(bool d3q19, int hidden, int prec, bool forced, int ncu, hipStream_t s,
                           const float* Ain, float* Aout, const float* theta, Grid G, Force Fc,
                           float rho0, float omega, float knn) {
  if (d3q19)
    return fwd_hidden<D3Q19>(hidden, prec, forced, ncu, s, Ain, Aout, theta, G, Fc, rho0, omega,
                             knn);
  return fwd_hidden<D2Q9>(hidden, prec, forced, ncu, s, Ain, Aout, theta, G, Fc, rho0, omega, knn);
}

}  // namespace lbm
