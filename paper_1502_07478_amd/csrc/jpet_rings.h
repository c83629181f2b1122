// The MLEM event pass on ring blocks: every wavefront works through blocks of its own and never waits for
// another wavefront between staging the region and flushing it.
//
// A block holds two events, one per half-wavefront, or one.  An event's ellipse lies in the lanes as
// RINGS rings of 32 (64) rows around its central row (see Plan), one row per lane and ring, the row's
// pixels in registers between the two passes.  Against the batch layout (jpet_binned.h, one row per
// thread, all events of a batch between two workgroup barriers) this leaves out the barriers, the
// LDS denominators and the per-wavefront reductions over rows of several events: one reduction over
// an event's lanes (in double precision, as between the wavefronts there) gives its denominator.
//
// Bound: VALU issue.  Per pixel the pass needs v_exp_f32, 3 FMAs for the exponent, P rho, D += P rho,
// and the scale and conversion of the back-projection; one LDS read and one LDS atomic go beside them.
#pragma once

#include <type_traits>

#include "jpet_rows.h"

namespace jpet {

namespace {

// A value that is the same in every lane, kept in a scalar register (the register cache leaves few
// vector registers for constants of the loop).
__device__ __forceinline__ float uniform_f(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// The lane's index, computed where it stands: two instructions instead of vector registers held
// through the loop for what follows from it.
__device__ __forceinline__ int fresh_lane() {
  int v;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(v));
  return v;
}

// A value the compiler knows nothing about.
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+s"(v));
  return v;
}

struct RingShared {
  unsigned zero, bad, odd;
};

// Accumulator units without a conversion.  A single-precision number up to 2^-125 is, bit for bit, the
// count of its 2^-149: with the image scaled by 2^-kBitsScale and the unit by 2^-149 on top, the product of
// pass 2 is the addend itself (at most 2^24 units), rounded to nearest.  Scaled so, the pixels' exp2(E) rho of an
// item whose image lies in [2^-66, 2^24) (or is 0) stay in the normal range: at least 2^-13 2^-66 2^-44.  The
// denominators need not: they carry kappa^-1/2, about sigma_z / (R sqrt 2).  Blocks with one below kBitsTiny,
// where 1 / D would leave the range, go pixel by pixel, with the image scaled up again.  Other
// images, and items of units finer than 2^-24 (fewer than 128 events), convert.  Ten iterations of 10M events on
// 400^2: 59.6 -> 58.5 ms, on 64 x 76: 22.3 -> 22.1.
constexpr int kBitsScale = 44, kBitsShift = 24;
constexpr float kBitsTiny = 0x1p-120f;

// Pass 1 along a lane's row of one ring: chunks below the
// wavefront's shortest row without masks, the others with the reads past the row's ends discarded
// (they stay inside the workgroup's LDS: the plan leaves H columns before the image and after the
// accumulators).
template <int H, int DEG>
__device__ __forceinline__ float ring_forward(const RowP& p, const float* __restrict__ rr, int pitch, int nl, int nr,
                                              int wminh, int wlh, float (&m)[2 * H]) {
  float D0 = 0.0f, D1 = 0.0f;
#pragma unroll
  for (int i0 = 0; i0 < H; i0 += 2) {
    constexpr int kStep = 2;
    if (i0 + kStep <= wminh && i0 + kStep <= H) {  // wavefront-uniform: every active lane's row is longer
      float lo[kStep], hi[kStep];
#pragma unroll
      for (int q = 0; q < kStep; ++q) {
        if (i0 + q >= H) continue;
        lo[q] = rr[(H - 1 - i0 - q) * pitch];
        hi[q] = rr[(H + i0 + q) * pitch];
      }
#pragma unroll
      for (int q = 0; q < kStep; ++q) {
        if (i0 + q >= H) continue;
        float el, eh;
        poly_pair<DEG>(p, i0 + q, el, eh);
        D0 += m[H - 1 - i0 - q] = el * lo[q];
        D1 += m[H + i0 + q] = eh * hi[q];
      }
    } else if (i0 < wlh) {  // wavefront-uniform
      float lo[kStep], hi[kStep];
#pragma unroll
      for (int q = 0; q < kStep; ++q) {
        if (i0 + q >= H) continue;
        lo[q] = rr[(H - 1 - i0 - q) * pitch];
        hi[q] = rr[(H + i0 + q) * pitch];
      }
#pragma unroll
      for (int q = 0; q < kStep; ++q) {
        if (i0 + q >= H) continue;
        float el, eh;
        poly_pair<DEG>(p, i0 + q, el, eh);
        D0 += m[H - 1 - i0 - q] = i0 + q < nl ? el * lo[q] : 0.0f;
        D1 += m[H + i0 + q] = i0 + q < nr ? eh * hi[q] : 0.0f;
      }
    } else {
#pragma unroll
      for (int q = 0; q < kStep; ++q) {
        if (i0 + q >= H) continue;
        m[H - 1 - i0 - q] = unread();
        m[H + i0 + q] = unread();
      }
    }
  }
  return D0 + D1;
}

// Pass 2 of one ring: m sc rounded into the fixed-point accumulators, up to the wavefront's longest
// row; past a row's own ends m is 0 and adds nothing.
template <int H, bool BITS>
__device__ __forceinline__ void ring_back(const float (&m)[2 * H], float sc, unsigned* __restrict__ a, int pitch,
                                          int wlh) {
  auto units = [&](float v) { return BITS ? __float_as_uint(v * sc) : (unsigned)fmaf(v, sc, 0.5f); };
#pragma unroll
  for (int i0 = 0; i0 < H; i0 += 2) {
    if (i0 < wlh) {  // wavefront-uniform
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (i0 + q >= H) continue;
        atomicAdd(&a[(H - 1 - i0 - q) * pitch], units(m[H - 1 - i0 - q]));
        atomicAdd(&a[(H + i0 + q) * pitch], units(m[H + i0 + q]));
      }
    }
  }
}

// A lane's row of one ring: the word's column and length.
struct RingRow {
  int rl, kc, nl, nr;  // region row, first pixel right of the centre, pixels on either side
};

__device__ __forceinline__ RingRow ring_row(uint32_t w16, int rl, int H) {
  const int len = (int)((w16 >> 8) & 127u);
  RingRow r;
  r.rl = len > 0 ? rl : 0;  // (an idle lane: row 0 of the region, and below the first columns)
  r.nl = len >> 1;
  r.nr = len - r.nl;
  r.kc = len > 0 ? (int)(w16 & 255u) + r.nl : H;
  return r;
}

// P at offset x from the row's centre, 0 (counted) where kappa <= 0.
__device__ __forceinline__ float exact_at(const RowF& k, float x, int* nbad) {
  const float kap = fmaf(x, k.dkap, k.kap0);
  if (!(kap > 0.0f)) {
    ++*nbad;
    return 0.0f;
  }
  const float rq = __builtin_amdgcn_rsqf(kap);
  const float tg = fmaf(x, k.dgs, k.gs0) * rq;
  return rq * __builtin_amdgcn_exp2f(fmaf(tg, tg, -fmaf(fmaf(k.qa, x, k.qb), x, k.qc)));
}

// The rings of a pair in turn, k counting up: f(k as a constant).
template <int K, int RINGS, class F>
__device__ __forceinline__ void each_ring(F&& f) {
  if constexpr (K < RINGS) {
    f(std::integral_constant<int, K>());
    each_ring<K + 1, RINGS>(f);
  }
}

template <int RINGS, int LEN>
struct RingCache {
  static constexpr int half(int k) { return ring_half_of(RINGS, LEN, k); }
  float m0[2 * half(0)], m1[2 * half(1)], m2[2 * half(2)], m3[2 * half(3)];
  template <int K>
  __device__ __forceinline__ auto& ring() {
    if constexpr (K == 0) return m0;
    else if constexpr (K == 1) return m1;
    else if constexpr (K == 2) return m2;
    else return m3;
  }
};

// One workgroup item (see event_pass_item in jpet_binned.h for the region and the units).  LDS: per
// wavefront two buffers of a block's constants (the next block's are copied in while this one runs),
// the column shift of every region row, then from p.lds_img the image and the accumulators, with
// p.slack columns free before and after them that masked reads and additions of 0 may touch.  FORWARD:
// the forward sums alone, to D_out (778k events on 400^2: 553 -> 425 us with the back-projection left out; 440 since
// the lanes' sums are added in double precision).
template <int RINGS, int LEN, bool SOLO, int PITCH, bool FORWARD = false>
__device__ __forceinline__ void ring_item(const Geo& g, const Plan& p, const unsigned char* __restrict__ blocks,
                                          const BinItem it, const float* __restrict__ rho,
                                          unsigned long long* __restrict__ acc, unsigned long long* __restrict__ cnt,
                                          unsigned char* smem, RingShared& ps, float* __restrict__ D_out) {
  constexpr int kEvents = SOLO ? 1 : 2, kHalf = WAVE / kEvents / 2;
  constexpr int kWords = (RINGS + 1) / 2;  // 32-bit words per lane: two rings each
  constexpr int kConst = kEvents * (int)sizeof(EvRow);
  constexpr int pitch = PITCH;
  const int npx = pitch * p.W;
  float* const rho_s = reinterpret_cast<float*>(smem + p.lds_img);
  unsigned* const acc_s = reinterpret_cast<unsigned*>(smem + p.lds_img) + npx;
  int* const off_s = reinterpret_cast<int*>(smem + p.lds_off);
  const int tid = threadIdx.x;
  const int lane = tid & (WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int waves = (int)(blockDim.x >> 6);
  const int nblk = (it.count + kEvents - 1) / kEvents;
  const unsigned char* const blk0 = blocks + (size_t)it.batch * (size_t)p.batch_bytes;
  unsigned char* const con_s = smem + wave * (2 * kConst);  // this wavefront's two buffers

  const int tz = it.bin % p.ntz;
  const int rest = it.bin / p.ntz;
  const int ty = rest % p.nty;
  const double tc = bin_slope(p, rest / p.nty);
  const int kmin = -max(shear_offset(g, tc, 0), shear_offset(g, tc, g.n_y - 1));
  const int rbase = ty * p.TY - p.HY;
  const int kbase = kmin + tz * p.TZ - p.HZ;

  // a block's constants (16 bytes per lane to LDS), words and ring tails
  uint32_t word[kWords];
  uint2 tails;
  auto fetch = [&](int q, int buf) {
    const unsigned char* blk = blk0 + (size_t)q * (size_t)p.batch_bytes;
    const int ln = fresh_lane();
    if (ln < kConst / 16)
      __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint4*>(blk + ln * 16),
                                       con_s + buf * kConst, 16, 0, 0);
#pragma unroll
    for (int j = 0; j < kWords; ++j)
      word[j] = reinterpret_cast<const uint32_t*>(blk + ring_words(kEvents, false))[j * WAVE + ln];
    tails = *reinterpret_cast<const uint2*>(blk + ring_tails(kEvents, false));
  };
  if (wave < nblk) fetch(wave, 0);
  if (tid == 0) ps.zero = ps.bad = ps.odd = 0u;
  for (int r = tid; r < p.RY; r += blockDim.x) off_s[r] = shear_offset(g, tc, rbase + r);
  bool bits = p.acc_shift <= kBitsShift;
  for (;;) {
    const float scale = bits ? __builtin_ldexpf(1.0f, -kBitsScale) : 1.0f;
    bool odd = false;
    __syncthreads();
    for (int cl = wave; cl < p.W; cl += waves) {
      const int kc = kbase + cl;
      for (int rl = lane; rl < pitch; rl += WAVE) {
        const int q = cl * pitch + rl;
        const int r = rbase + rl;
        float v = 0.0f;
        if (rl < p.RY && r >= 0 && r < g.n_y) {
          const int k = kc + off_s[rl];
          if (k >= 0 && k < g.n_z) v = rho[(int64_t)r * g.n_z + k];
        }
        odd |= v != 0.0f && !(v >= __builtin_ldexpf(1.0f, -66) && v < 16777216.0f);
        rho_s[q] = fmaf(v, scale, 0.0f);  // (and -0 as 0: its bits would be 2^31 units)
        if constexpr (!FORWARD) acc_s[q] = 0u;
      }
    }
    if (bits && odd) ps.odd = 1u;
    __syncthreads();
    if (!bits || ps.odd == 0u) break;  // uniform over the workgroup
    bits = false;                      // once more, as it is
  }
  const float kUnit = uniform_f(__builtin_ldexpf(1.0f, bits ? p.acc_shift - 149 : p.acc_shift));
  const float tiny = uniform_f(bits ? kBitsTiny : 1e-28f);

  int buf = 0;
  for (int q = wave; q < nblk; q += waves, buf ^= 1) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this block's constants, words and tails have arrived
    const int ln = fresh_lane(), l = ln & (2 * kHalf - 1);
    const int lrow = l - kHalf, lstep = l < kHalf ? -kHalf : kHalf;  // the lane's row in ring k: lrow + k lstep
    const EvRow& c = reinterpret_cast<const EvRow*>(con_s + buf * kConst)[SOLO ? 0 : ln >> 5];
    // ring tails (uniform): longest and shortest row, how the rows are evaluated
    const uint32_t t01 = __builtin_amdgcn_readfirstlane(tails.x), t23 = __builtin_amdgcn_readfirstlane(tails.y);
    uint32_t w[kWords];
#pragma unroll
    for (int j = 0; j < kWords; ++j) w[j] = word[j];
    if (q + waves < nblk) fetch(q + waves, buf ^ 1);

    // an event's denominator (on one of its lanes)
    auto denominator = [&](double D) {
      if (c.index < 0) return;  // no event
      if (!(D > 0.0)) atomicAdd(&ps.zero, 1u);
      if constexpr (FORWARD) D_out[c.index] = (float)(D * g.cnorm * (bits ? __builtin_ldexp(1.0, kBitsScale) : 1.0));
    };
    auto tail = [&](int k) { return ((k < 2 ? t01 : t23) >> (16 * (k & 1))) & 0xffffu; };
    auto row = [&](int k, int H) { return ring_row(w[k >> 1] >> (16 * (k & 1)), c.mid + lrow + k * lstep, H); };
    // the sum over an event's lanes, to all of them: of the lanes' single-precision sums over their rows, in double
    // precision, so that a denominator is rounded no more often than its rows are
    auto event_sum = [&](float v, double& lo, double& hi) {
      if constexpr (SOLO) {
        lo = hi = wave_sum_dpp_d((double)v);
        return lo;
      } else {
        const double h = half_sums_dpp_d((double)v);
        lo = lane_value_d(h, 31);
        hi = lane_value_d(h, 63);
        return ln < 32 ? lo : hi;
      }
    };
    if ((t01 >> 14 & 3u) != kRowExact) {
      RingCache<RINGS, LEN> cache;
      float F[RINGS];
      int at[RINGS];  // cache slot 0 of the lane's row in the region, kNoRow for no row
      constexpr int kNoRow = -(1 << 30);
      float D = 0.0f;
      each_ring<0, RINGS>([&](auto kk) {
        constexpr int k = kk, H = ring_half_of(RINGS, LEN, k);
        const uint32_t tw = tail(k);
        const int wlh = (int)((tw & 127u) + 1) >> 1, wminh = (int)((tw >> 7) & 127u) >> 1;
        const RingRow r = row(k, H);
        const RowF rk = ring_constants(c, (float)(lrow + k * lstep), r.kc + off_s[r.rl]);
        at[k] = (r.kc - H) * pitch + r.rl;
        const float* const rr = rho_s + at[k];
        RowP rp;
        float S;
        if ((tw >> 14) == kRowPoly5) {
          F[k] = row_poly<5>(rk, (float)r.nr - 0.5f, rp);
          S = ring_forward<H, 5>(rp, rr, pitch, r.nl, r.nr, wminh, wlh, cache.template ring<k>());
        } else {
          F[k] = row_poly<6>(rk, (float)r.nr - 0.5f, rp);
          S = ring_forward<H, 6>(rp, rr, pitch, r.nl, r.nr, wminh, wlh, cache.template ring<k>());
        }
        if (r.nr > 0) D = fmaf(F[k], S, D);
        else at[k] = kNoRow;
      });
      double Dlo, Dhi;
      const double De = event_sum(D, Dlo, Dhi);  // the event's denominator
      // (a unit / D overflows a float only for D < 1e-28, its reciprocal vanishes above 2^126, and rows without their
      // factor F overflow first: such blocks take the way below)
      auto plain = [&](float v) { return v <= 0.0f || (v >= tiny && v <= 0x1p126f); };
      if (plain((float)Dlo) && plain((float)Dhi)) {  // wavefront-uniform
        if (l == 0) denominator(De);
        if constexpr (FORWARD) continue;
        const float sc = De > 0.0 ? kUnit * __builtin_amdgcn_rcpf((float)De) : 0.0f;
        each_ring<0, RINGS>([&](auto kk) {
          constexpr int k = kk, H = ring_half_of(RINGS, LEN, k);
          const int wlh = (int)((tail(k) & 127u) + 1) >> 1;
          if (at[k] != kNoRow && sc > 0.0f) {
            if (bits) ring_back<H, true>(cache.template ring<k>(), sc * F[k], acc_s + at[k], pitch, wlh);
            else ring_back<H, false>(cache.template ring<k>(), sc * F[k], acc_s + at[k], pitch, wlh);
          }
        });
        continue;
      }
    }

    // pixel by pixel, evaluated in both passes; P rho scaled by 2^64 against overflow of unit / D for D below 1 (P rho
    // is below D), and in D too where the image is scaled down.
    // (Rolled, and with the constants read again: shared with the way above they would take 26 vector
    // registers through it.)
    asm volatile("" ::: "memory");
    float D = 0.0f;
    int nbad = 0, again = 0;
    const int first = opaque(0);
    const float up = bits ? 18446744073709551616.0f : 1.0f;
    for (int k = first; k < RINGS; ++k) {
      const RingRow r = row(k, 0);
      const RowF rk = ring_constants(c, (float)(lrow + k * lstep), r.kc + off_s[r.rl]);
      for (int j = -r.nl; j < r.nr; ++j)
        D = fmaf(exact_at(rk, (float)j + 0.5f, &nbad), rho_s[(r.kc + j) * pitch + r.rl] * up, D);
    }
    if (nbad) atomicAdd(&ps.bad, (unsigned)nbad);
    double Dlo, Dhi;
    const double De = event_sum(D, Dlo, Dhi) / up;
    if (l == 0) denominator(De);
    if (FORWARD || !(De > 0.0)) continue;
    const float lift = De < 1.0 ? 18446744073709551616.0f : 1.0f;
    const float sc = (float)(__builtin_ldexp(1.0, p.acc_shift) / (De * lift));
    for (int k = first; k < RINGS; ++k) {
      const RingRow r = row(k, 0);
      const RowF rk = ring_constants(c, (float)(lrow + k * lstep), r.kc + off_s[r.rl]);
      for (int j = -r.nl; j < r.nr; ++j) {
        const int px = (r.kc + j) * pitch + r.rl;
        const float m = exact_at(rk, (float)j + 0.5f, &again) * rho_s[px] * lift;
        atomicAdd(&acc_s[px], (unsigned)fmaf(m, sc, 0.5f));
      }
    }
  }
  __syncthreads();

  // add the region's accumulators to the global image.  Lanes run along the image's rows, so that a
  // wavefront's 64-bit atomics fall into a few lines; the LDS reads then meet in a bank, which costs
  // less (lanes along the region's columns, free of conflicts: every atomic a line of its own)
  const int flush_shift = 32 - p.acc_shift;
  const float inv_w = 1.0f / (float)p.W;
  for (int q = FORWARD ? p.RY * p.W : tid; q < p.RY * p.W; q += (int)blockDim.x) {
    const int rl = (int)(((float)q + 0.5f) * inv_w), cl = q - rl * p.W;
    const unsigned long long a = (unsigned long long)acc_s[cl * pitch + rl] << flush_shift;
    if (a == 0ull) continue;
    const int r = rbase + rl;
    const int k = kbase + cl + off_s[rl];
    if (r >= 0 && r < g.n_y && k >= 0 && k < g.n_z) atomicAdd(&acc[(int64_t)r * g.n_z + k], a);
  }
  if (tid == 0) {
    if (ps.zero) atomicAdd(&cnt[C_ZERO_DEN], (unsigned long long)ps.zero);
    if (ps.bad) atomicAdd(&cnt[C_KAPPA_BAD], (unsigned long long)ps.bad);
  }
}

template <int SHAPE, int PITCH, bool FORWARD>
__global__ void __launch_bounds__((shape_threads(SHAPE)), (shape_waves_per_simd(SHAPE)))
    k_event_pass_rings(Geo g, Plan p, const unsigned char* __restrict__ blocks, const BinItem* __restrict__ items,
                       const float* __restrict__ rho, unsigned long long* __restrict__ acc,
                       unsigned long long* __restrict__ cnt, float* __restrict__ D_out) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ RingShared ps;
  if ((unsigned long long)blockIdx.x >= cnt[C_ITEMS]) return;  // uniform over the workgroup
  ring_item<shape_rings(SHAPE), shape_len(SHAPE), (SHAPE >= 1000), PITCH, FORWARD>(g, p, blocks, items[blockIdx.x],
                                                                                   rho, acc, cnt, smem, ps, D_out);
}

// The same over a class of a batch's instances (see k_event_pass_batched in jpet_binned.h).
template <int SHAPE, int PITCH>
__global__ void __launch_bounds__((shape_threads(SHAPE)), (shape_waves_per_simd(SHAPE)))
    k_event_pass_rings_batched(const BatchInst* __restrict__ inst, int count, unsigned total) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ RingShared ps;
  const unsigned w = blockIdx.x;
  if (w >= total) return;  // uniform over the workgroup
  int lo = 0, hi = count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (inst[mid].item_begin <= (int64_t)w) lo = mid;
    else hi = mid - 1;
  }
  const BatchInst& I = inst[lo];
  const BinItem it = I.items[(int64_t)w - I.item_begin];
  ring_item<shape_rings(SHAPE), shape_len(SHAPE), (SHAPE >= 1000), PITCH>(I.g, I.p, I.blocks, it, I.rho, I.acc, I.cnt,
                                                                          smem, ps, nullptr);
}

}  // namespace

template <int SHAPE>
hipError_t Rings<SHAPE>::event_pass(const Geo& g, const Plan& p, const Workspace& ws, const float* rho, float* D_out,
                                    hipStream_t st) {
  if (p.pitch != shape_pitch(SHAPE, 0) && p.pitch != shape_pitch(SHAPE, 1)) return hipErrorInvalidValue;
  constexpr int kFirst = shape_pitch(SHAPE, 0), kSecond = shape_pitch(SHAPE, 1);
  auto kern = p.pitch == kFirst ? (D_out ? k_event_pass_rings<SHAPE, kFirst, true>
                                         : k_event_pass_rings<SHAPE, kFirst, false>)
                                : (D_out ? k_event_pass_rings<SHAPE, kSecond, true>
                                         : k_event_pass_rings<SHAPE, kSecond, false>);
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kRingLdsLimit);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)p.max_items), dim3(64 * p.waves), p.lds_bytes, st, g, p, ws.batches,
                     ws.items, rho, ws.acc, ws.cnt, D_out);
  return hipGetLastError();
}

template <int SHAPE>
hipError_t Rings<SHAPE>::batched(const BatchInst* table, int count, int waves, int pitch, unsigned items,
                                 size_t lds_bytes, hipStream_t st) {
  // the dynamic LDS limit is raised beforehand (set_batched_lds), outside any stream capture
  if (pitch != shape_pitch(SHAPE, 0) && pitch != shape_pitch(SHAPE, 1)) return hipErrorInvalidValue;
  auto kern = pitch == shape_pitch(SHAPE, 0) ? k_event_pass_rings_batched<SHAPE, shape_pitch(SHAPE, 0)>
                                             : k_event_pass_rings_batched<SHAPE, shape_pitch(SHAPE, 1)>;
  hipLaunchKernelGGL(kern, dim3(items), dim3(64 * waves), lds_bytes, st, table, count, items);
  return hipGetLastError();
}

template <int SHAPE>
const void* Rings<SHAPE>::batched_kernel(int, int pitch) {
  return pitch == shape_pitch(SHAPE, 0)   ? (const void*)k_event_pass_rings_batched<SHAPE, shape_pitch(SHAPE, 0)>
         : pitch == shape_pitch(SHAPE, 1) ? (const void*)k_event_pass_rings_batched<SHAPE, shape_pitch(SHAPE, 1)>
                                          : nullptr;
}

}  // namespace jpet
