// Event passes without binning (one wavefront or one thread per event), the pixel update (Eq. 3/5), the
// batch's table, and the dispatch of the binned passes (jpet_binned.h) by register cache.
#include "jpet_device.h"

namespace jpet {

namespace {

// Generic pass for geometries whose rows or regions do not fit the tiled pass: one wavefront per
// event, one lane per row, kernel values recomputed in pass 2, fixed-point global atomics.
__global__ void __launch_bounds__(256) k_event_pass_generic(Geo g, int64_t n, const EventRec* __restrict__ ev,
                                                            const float* __restrict__ rho,
                                                            unsigned long long* __restrict__ acc,
                                                            unsigned long long* __restrict__ cnt,
                                                            float* __restrict__ D_out) {
  const int lane = threadIdx.x & (WAVE - 1);
  const int64_t j = (int64_t)blockIdx.x * (blockDim.x / WAVE) + (threadIdx.x / WAVE);
  if (j >= n) return;
  const EventRec e = ev[j];
  if (e.r1 < e.r0) return;
  int nbad = 0;  // pixels of this lane's row with kappa <= 0 (P := 0)
  float D = 0.0f;
  for (int b0 = e.r0; b0 <= e.r1; b0 += WAVE) {
    const int i = b0 + lane;
    int klo, khi;
    if (i <= e.r1 && row_interval(g, e, i, &klo, &khi)) {
      double kf, ks;
      const RowK r = row_constants(g, e, i, klo, &kf, &ks);
      const float* rr = rho + (int64_t)i * g.n_z;
      for (int k = klo; k <= khi; ++k) D += kernel_guarded(r, (float)(k - klo), &nbad) * rr[k];
    }
  }
  D = wave_sum(D);
  const unsigned long long nbad_w = wave_sum_u64((unsigned long long)nbad);
  if (lane == 0 && nbad_w) atomicAdd(&cnt[C_KAPPA_BAD], nbad_w);
  int again = 0;  // pass 2 recomputes the same values: not counted twice
  if (lane == 0 && D_out) D_out[j] = (float)((double)D * g.cnorm);
  if (!(D > 0.0f)) {
    if (lane == 0) atomicAdd(&cnt[C_ZERO_DEN], 1ull);
    return;
  }
  const float sc = (float)(4294967296.0 / (double)D);
  for (int b0 = e.r0; b0 <= e.r1; b0 += WAVE) {
    const int i = b0 + lane;
    int klo, khi;
    if (i <= e.r1 && row_interval(g, e, i, &klo, &khi)) {
      double kf, ks;
      const RowK r = row_constants(g, e, i, klo, &kf, &ks);
      const float* rr = rho + (int64_t)i * g.n_z;
      unsigned long long* aa = acc + (int64_t)i * g.n_z;
      for (int k = klo; k <= khi; ++k) {
        const float m = kernel_guarded(r, (float)(k - klo), &again) * rr[k];
        if (m > 0.0f) atomicAdd(&aa[k], (unsigned long long)(unsigned)fmaf(m, sc, 0.5f));
      }
    }
  }
}

// Thread-granularity pass (comparison only): one thread per event walks every pixel of its
// ellipse twice, first for D, then adding the back-projection with global fixed-point atomics.
// This is the GPU work split the paper measures as its "thread" variant (Sec. 4, Table 1); lanes
// of a wavefront hold events of different sizes and read unrelated image rows.
__global__ void __launch_bounds__(256) k_event_pass_thread(Geo g, int64_t n, const EventRec* __restrict__ ev,
                                                           const float* __restrict__ rho,
                                                           unsigned long long* __restrict__ acc,
                                                           unsigned long long* __restrict__ cnt,
                                                           float* __restrict__ D_out) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  const EventRec e = ev[j];
  if (e.r1 < e.r0) return;
  int nbad = 0;  // pixels of this event with kappa <= 0 (P := 0)
  float D = 0.0f;
  for (int i = e.r0; i <= e.r1; ++i) {
    int klo, khi;
    if (!row_interval(g, e, i, &klo, &khi)) continue;
    double kf, ks;
    const RowK r = row_constants(g, e, i, klo, &kf, &ks);
    const float* rr = rho + (int64_t)i * g.n_z;
    for (int k = klo; k <= khi; ++k) D += kernel_guarded(r, (float)(k - klo), &nbad) * rr[k];
  }
  if (nbad) atomicAdd(&cnt[C_KAPPA_BAD], (unsigned long long)nbad);
  int again = 0;  // pass 2 recomputes the same values: not counted twice
  if (D_out) D_out[j] = (float)((double)D * g.cnorm);
  if (!(D > 0.0f)) {
    atomicAdd(&cnt[C_ZERO_DEN], 1ull);
    return;
  }
  const float sc = (float)(4294967296.0 / (double)D);
  for (int i = e.r0; i <= e.r1; ++i) {
    int klo, khi;
    if (!row_interval(g, e, i, &klo, &khi)) continue;
    double kf, ks;
    const RowK r = row_constants(g, e, i, klo, &kf, &ks);
    const float* rr = rho + (int64_t)i * g.n_z;
    unsigned long long* aa = acc + (int64_t)i * g.n_z;
    for (int k = klo; k <= khi; ++k) {
      const float m = kernel_guarded(r, (float)(k - klo), &again) * rr[k];
      if (m > 0.0f) atomicAdd(&aa[k], (unsigned long long)(unsigned)fmaf(m, sc, 0.5f));
    }
  }
}

// rho_l = acc_l 2^-32 / s_l (0 where s_l = 0), or acc_l 2^-32 without sensitivity; acc cleared.
// cnt (nullable): the pass's counters, cleared for the next one.
__global__ void k_update(int64_t npix, const float* __restrict__ s, float* __restrict__ rho,
                         unsigned long long* __restrict__ acc, unsigned long long* __restrict__ cnt) {
  if (cnt && blockIdx.x == 0 && threadIdx.x == 0) cnt[C_ZERO_DEN] = cnt[C_KAPPA_BAD] = 0ull;
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < npix; q += (int64_t)gridDim.x * blockDim.x) {
    const double a = (double)acc[q] * 2.3283064365386962890625e-10;
    double v;
    if (s) {
      const float sv = s[q];
      v = sv > 0.0f ? a / (double)sv : 0.0;
    } else {
      v = a;
    }
    rho[q] = (float)v;
    acc[q] = 0ull;
  }
}

__global__ void k_write_insts(InstWrite w, BatchInst* __restrict__ table) {
  const int t = threadIdx.x;
  if (t < w.count) table[w.first + t] = w.v[t];
}

// per-iteration counters of every instance: zero-denominator events, non-positive kappa pairs
__global__ void k_batched_reset(const BatchInst* __restrict__ table, int count) {
  for (int k = threadIdx.x; k < count; k += blockDim.x) {
    table[k].cnt[C_ZERO_DEN] = 0ull;
    table[k].cnt[C_KAPPA_BAD] = 0ull;
  }
}

// rho = acc 2^-32 / s of every instance (blockIdx.y: table entry)
__global__ void k_update_batched(const BatchInst* __restrict__ table) {
  const BatchInst& I = table[blockIdx.y];
  const int64_t npix = (int64_t)I.g.n_y * I.g.n_z;
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < npix; q += (int64_t)gridDim.x * blockDim.x) {
    const double a = (double)I.acc[q] * 2.3283064365386962890625e-10;
    double v;
    if (I.s) {
      const float sv = I.s[q];
      v = sv > 0.0f ? a / (double)sv : 0.0;
    } else {
      v = a;
    }
    I.rho[q] = (float)v;
    I.acc[q] = 0ull;
  }
}

// the binned passes compiled for a plan's register cache (pass_kernel)
template <int K, class F>
hipError_t by_shape(int shape, F f) {
  if constexpr (K < (int)(sizeof(kRingShapes) / sizeof(kRingShapes[0]))) {
    return shape == kRingShapes[K] ? f(Rings<kRingShapes[K]>()) : by_shape<K + 1>(shape, f);
  } else {
    return hipErrorInvalidValue;
  }
}

template <class F>
hipError_t by_cache(int kernel, F f) {
  switch (kernel) {
    case 16: return f(Binned<16>());
    case 32: return f(Binned<32>());
    case 48: return f(Binned<48>());
    case 64: return f(Binned<64>());
    default: return hipErrorInvalidValue;
  }
}

template <class F>
hipError_t by_kernel(int kernel, F f) {
  return kernel > 10000 ? by_shape<0>(kernel - 10000, f) : by_cache(kernel, f);
}

}  // namespace

hipError_t launch_loglik_tiled(const Geo& g, const Plan& p, int64_t n, const Workspace& ws, const float* rho,
                               float* D_out, bool value_only, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (p.rings) {
    if (value_only) return launch_loglik_rings_value(g, p, ws, rho, D_out, st);
    return by_shape<0>(pass_kernel(p) - 10000, [&](auto b) { return b.loglik(g, p, ws, rho, D_out, st); });
  }
  return by_cache(p.maxlen, [&](auto b) { return b.loglik(g, p, ws, rho, D_out, value_only, st); });
}

hipError_t launch_write_insts(const InstWrite& w, BatchInst* table, hipStream_t st) {
  hipLaunchKernelGGL(k_write_insts, dim3(1), dim3(64), 0, st, w, table);
  return hipGetLastError();
}

hipError_t launch_batched_reset(const BatchInst* table, int count, hipStream_t st) {
  hipLaunchKernelGGL(k_batched_reset, dim3(1), dim3(256), 0, st, table, count);
  return hipGetLastError();
}

hipError_t launch_event_pass_batched(const BatchInst* table, int count, int kernel, int waves, int pitch,
                                     size_t lds_bytes, int64_t items, hipStream_t st) {
  if (count <= 0 || items <= 0) return hipSuccess;
  if (items > 0x7fffffffll) return hipErrorInvalidValue;
  return by_kernel(kernel, [&](auto b) { return b.batched(table, count, waves, pitch, (unsigned)items, lds_bytes, st); });
}

hipError_t set_batched_lds(int kernel, int waves, int pitch, size_t lds_bytes) {
  return by_kernel(kernel, [&](auto b) {
    const void* f = b.batched_kernel(waves, pitch);
    if (!f) return hipErrorInvalidValue;  // not compiled for this pitch
    return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kernel > 10000 ? kRingLdsLimit : (int)lds_bytes);
  });
}

hipError_t launch_update_batched(const BatchInst* table, int count, int64_t max_npix, hipStream_t st) {
  if (count <= 0 || max_npix <= 0) return hipSuccess;
  int64_t bx = (max_npix + 255) / 256;
  if (bx > 1024) bx = 1024;
  hipLaunchKernelGGL(k_update_batched, dim3((unsigned)bx, (unsigned)count), dim3(256), 0, st, table);
  return hipGetLastError();
}

hipError_t launch_event_pass(const Geo& g, const Plan& p, int64_t n, const Workspace& ws, const float* rho,
                             hipStream_t st, int granularity, float* D_out) {
  if (n <= 0) return hipSuccess;
  if (granularity == kPassThreadPerEvent) {
    const int64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(k_event_pass_thread, dim3((unsigned)blocks), dim3(256), 0, st, g, n, ws.ev, rho, ws.acc, ws.cnt,
                       D_out);
    return hipGetLastError();
  }
  if (p.tiled && granularity == kPassPlanned) {
    return by_kernel(pass_kernel(p), [&](auto b) { return b.event_pass(g, p, ws, rho, D_out, st); });
  }
  const int64_t blocks = (n + 3) / 4;
  hipLaunchKernelGGL(k_event_pass_generic, dim3((unsigned)blocks), dim3(256), 0, st, g, n, ws.ev, rho, ws.acc, ws.cnt,
                     D_out);
  return hipGetLastError();
}

hipError_t launch_update(const Geo& g, const float* s, float* rho, const Workspace& ws, hipStream_t st) {
  const int64_t npix = (int64_t)g.n_y * g.n_z;
  int64_t blocks = (npix + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_update, dim3((unsigned)blocks), dim3(256), 0, st, npix, s, rho, ws.acc,
                     ws.more ? ws.cnt : nullptr);
  return hipGetLastError();
}

}  // namespace jpet
