// The log-likelihood's value on ring blocks: one kernel per number of rings, whatever their rows' length.
#include "jpet_rings_loglik.h"

namespace jpet {

namespace {

template <int RINGS, bool SOLO>
__global__ void __launch_bounds__(1024, 6)
    k_loglik_rings_value(Geo g, Plan p, const unsigned char* __restrict__ blocks, const BinItem* __restrict__ items,
                         const float* __restrict__ rho, float* __restrict__ D_out, double* __restrict__ red,
                         unsigned long long* __restrict__ cnt, const int32_t* __restrict__ order) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ LogShared ps;
  if ((unsigned long long)blockIdx.x >= cnt[C_ITEMS]) return;  // uniform over the workgroup
  loglik_item<RINGS, 2, SOLO, 0, true>(g, p, blocks, items[blockIdx.x], rho, nullptr, D_out, red, cnt, order, smem, ps);
}

}  // namespace

hipError_t launch_loglik_rings_value(const Geo& g, const Plan& p, const Workspace& ws, const float* rho, float* D_out,
                                     hipStream_t st) {
  auto kern = p.solo ? (p.rings == 1   ? k_loglik_rings_value<1, true>
                        : p.rings == 2 ? k_loglik_rings_value<2, true>
                        : p.rings == 3 ? k_loglik_rings_value<3, true>
                                       : k_loglik_rings_value<4, true>)
                     : (p.rings == 1   ? k_loglik_rings_value<1, false>
                        : p.rings == 2 ? k_loglik_rings_value<2, false>
                                       : k_loglik_rings_value<3, false>);
  // the image alone, with the slack after it
  const size_t lds = (size_t)p.lds_img + 4u * (size_t)p.pitch * (size_t)(p.W + p.slack);
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kRingLdsLimit);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)p.max_items), dim3(64 * p.waves), lds, st, g, p, ws.batches, ws.items, rho,
                     D_out, ws.red, ws.cnt, ws.order);
  return hipGetLastError();
}

}  // namespace jpet
