// The log-likelihood passes on ring blocks (see jpet_rings.h for the blocks and the work split).
//
// With E(x) the exponent of a row's polynomial form and v = P' rho, the derivatives of log D with respect
// to u and w need four sums over a row's pixels (RowD in jpet_binned.h): S0 = sum v, X = sum v (exponent),
// G = sum v sqrt(S) gamma^ / kappa and H = sum v (1/kappa + (gamma^/kappa)^2).  Along a row kappa is
// kappa_0 (1 + delta x), so all four are combinations of the moments M_k = sum v x^k, k <= 5 (6 for
// kRowPoly6), with 1 / (1 + delta x) expanded as in the exponent.  The pixels at x and -x share the powers:
// v+ + v- goes into the even moments and v+ - v- into the odd ones, 4 (4.5) VALU operations per pixel
// with S0 among them, against 8 for the sums pixel by pixel.
//
// Bound by VALU issue, as the event pass is.  1M events, 977M pairs on 200^2 of 2.5 mm (shape 318): 1.81 ms
// with the sums pixel by pixel on the former batches, 0.94 ms here (1.0e12 pairs/s).  A call for the
// value alone, 400k prepared events on the same grid: 467 us and 214.
#pragma once

#include <type_traits>

#include "jpet_rings.h"

namespace jpet {

namespace {

// The moments of one row.
template <int DEG>
struct Moments {
  float m[7] = {};
  // the pixels at x = -(i + 1/2) and i + 1/2
  __device__ __forceinline__ void add(int i, float lo, float hi) {
    const float x = (float)i + 0.5f, X = x * x;
    const float s = hi + lo, d = hi - lo;
    m[0] += s;
    m[1] = fmaf(d, x, m[1]);
    m[2] = fmaf(s, X, m[2]);
    m[3] = fmaf(d, x * X, m[3]);
    m[4] = fmaf(s, X * X, m[4]);
    m[5] = fmaf(d, x * X * X, m[5]);
    if constexpr (DEG == 6) m[6] = fmaf(s, X * X * X, m[6]);
  }
};

// Geometry constants of the derivatives, in scalar registers.
struct LogGeo {
  float pix, fa, qlo;  // qlo: see row_poly
};

// A row's parts of the derivatives of log D with respect to u and w, from S0, X, G, H (see RowD); x: the row from its
// event's central row on.  With A and B their sums over an event's rows,
//   D_u / D = cu - 1 / (2 u) + A / (2 S u D),  D_w / D = cw - B / (2 S w D),
// whose constants are applied in double precision, event by event: what they multiply cancels to a few percent over the
// events, and a constant rounded to 2^-25 would leave its share in every one of them.  The constants inside A and B
// multiply terms of some percent of the others.
__device__ __forceinline__ void row_derivatives(const EvRow& c, const EvLog& q, float x, const LogGeo& g,
                                                float S0, float X, float G, float H, float& A, float& B) {
  const float irs = 1.1774100225154747f;  // 1 / sqrt(log2(e) / 2)
  const float S2 = 1.4426950408889634f;   // log2(e)
  const float Y = fmaf(x, g.pix, q.Y0), dy = fmaf(x, g.pix, -q.yr);
  const float wKl = Y * fmaf(q.A2, Y, q.A3 * dy);
  const float cr = fmaf(q.GK, fmaf(g.fa, Y, 2.0f * dy), wKl);
  const float er = irs * fmaf(fmaf(c.S2, x, c.S1), x, c.S0);
  const float wGl = fmaf(-q.GG, dy, er);
  const float SwBl = fmaf(fmaf(c.Q2, x, c.Q1), x, c.Q0);
  A = fmaf(SwBl, S0, fmaf(S2, fmaf(-irs * er, G, 0.5f * cr * H), X));
  B = fmaf(SwBl, S0, -S2 * fmaf(irs * wGl, G, -0.5f * wKl * H));
}

// X, G and H of a row from its moments.
template <int DEG>
__device__ __forceinline__ void row_sums(const RowF& k, const Moments<DEG>& M, float& X, float& G, float& H) {
  const float iS = 1.3862943611198906f;
  const float rq = __builtin_amdgcn_rsqf(k.kap0), rk = rq * rq, dl = k.dkap * rk;
  const float h0 = k.gs0 * rq, h1 = k.dgs * rq, d = fmaf(-dl, h0, h1), w = d * d;
  const float A = k.gs0, B = fmaf(-k.gs0, dl, k.dgs);  // (gs0 + dgs x) / (1 + dl x) = A + B x / (1 + dl x)
  const float* const m = M.m;
  // sums of v x / (1 + dl x), v x^2 / (1 + dl x) and v x^2 / (1 + dl x)^2
  float t5 = m[5], j2 = fmaf(-4.0f * dl, m[5], 3.0f * m[4]);
  if constexpr (DEG == 6) {
    t5 = fmaf(-dl, m[6], m[5]);
    j2 = fmaf(-dl, fmaf(-5.0f * dl, m[6], 4.0f * m[5]), 3.0f * m[4]);
  }
  const float t4 = fmaf(-dl, t5, m[4]), t3 = fmaf(-dl, t4, m[3]), t2 = fmaf(-dl, t3, m[2]), j1 = fmaf(-dl, t2, m[1]);
  j2 = fmaf(dl, fmaf(dl, j2, -2.0f * m[3]), m[2]);
  const float i1 = fmaf(-dl, j1, m[0]);
  X = fmaf(fmaf(h0, h0, -k.qc), m[0], fmaf(fmaf(h0, h1 + d, -k.qb), m[1], fmaf(-k.qa, m[2], w * t2)));
  G = rk * fmaf(A, m[0], B * j1);
  H = rk * fmaf(iS * rk, fmaf(A * A, m[0], fmaf(2.0f * A * B, j1, B * B * j2)), i1);
}

// Pass 1 along a row: exp2(E) into the cache, the moments of exp2(E) rho (see ring_forward).
template <int H, int DEG>
__device__ __forceinline__ void ring_moments(const RowP& p, const float* __restrict__ rr, int pitch, int nl, int nr,
                                             int wminh, int wlh, float (&m)[2 * H], Moments<DEG>& M) {
#pragma unroll
  for (int i0 = 0; i0 < H; i0 += 2) {
    if (i0 + 2 <= wminh && i0 + 2 <= H) {  // wavefront-uniform: every active lane's row is longer
      float lo[2], hi[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        lo[q] = rr[(H - 1 - i0 - q) * pitch];
        hi[q] = rr[(H + i0 + q) * pitch];
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        poly_pair<DEG>(p, i0 + q, m[H - 1 - i0 - q], m[H + i0 + q]);
        M.add(i0 + q, m[H - 1 - i0 - q] * lo[q], m[H + i0 + q] * hi[q]);
      }
    } else if (i0 < wlh) {  // wavefront-uniform
      float lo[2], hi[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (i0 + q >= H) continue;
        lo[q] = rr[(H - 1 - i0 - q) * pitch];
        hi[q] = rr[(H + i0 + q) * pitch];
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (i0 + q >= H) continue;
        poly_pair<DEG>(p, i0 + q, m[H - 1 - i0 - q], m[H + i0 + q]);
        // (past a row's end the reads may fall into the region's doubles)
        M.add(i0 + q, i0 + q < nl ? m[H - 1 - i0 - q] * lo[q] : 0.0f, i0 + q < nr ? m[H + i0 + q] * hi[q] : 0.0f);
      }
    } else {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (i0 + q >= H) continue;
        m[H - 1 - i0 - q] = unread();
        m[H + i0 + q] = unread();
      }
    }
  }
}

// Pass 2 along a row: B += P / D in the region's doubles, the row's own pixels only.
template <int H>
__device__ __forceinline__ void ring_back_f64(const float (&m)[2 * H], float sc, double* __restrict__ b, int pitch,
                                              int nl, int nr, int wminh, int wlh) {
  auto add = [&](int slot) { unsafeAtomicAdd(&b[slot * pitch], (double)(m[slot] * sc)); };
#pragma unroll
  for (int i0 = 0; i0 < H; i0 += 2) {
    if (i0 + 2 <= wminh && i0 + 2 <= H) {  // wavefront-uniform
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        add(H - 1 - i0 - q);
        add(H + i0 + q);
      }
    } else if (i0 < wlh) {  // wavefront-uniform
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (i0 + q >= H) continue;
        if (i0 + q < nl) add(H - 1 - i0 - q);
        if (i0 + q < nr) add(H + i0 + q);
      }
    }
  }
}

// One row of the value's forward sum, rolled: no cache, so one kernel serves every row length.
template <int DEG>
__device__ __forceinline__ float ring_value(const RowP& p, const float* __restrict__ rr, int pitch, int nl, int nr,
                                            int wlh) {
  float D0 = 0.0f, D1 = 0.0f, x = 0.5f;
  const float *lo = rr - pitch, *hi = rr;
#pragma unroll 2
  for (int i = 0; i < wlh; ++i) {
    // (an idle lane reads on from its own place: it stays where the wavefront's rows do)
    const float rl = *lo, rh = *hi;
    const float X = x * x;
    float ev = fmaf(p.c4, X, p.c2);
    if constexpr (DEG == 6) ev = fmaf(fmaf(p.c6, X, p.c4), X, p.c2);
    ev *= X;
    const float od = fmaf(fmaf(p.c5, X, p.c3), X, p.c1);
    const float el = __builtin_amdgcn_exp2f(fmaf(od, -x, ev)), eh = __builtin_amdgcn_exp2f(fmaf(od, x, ev));
    D0 += i < nl ? el * rl : 0.0f;
    D1 += i < nr ? eh * rh : 0.0f;
    lo -= pitch;
    hi += pitch;
    x += 1.0f;
  }
  return D0 + D1;
}

constexpr float kFloatMax = 3.402823466e38f;

struct LogShared {
  unsigned zero, bad;
  double sum[3];
};

// One item.  LDS: as in the pass on ring blocks, but for the accumulators: doubles, or none for the VALUE
// alone; before the image, from p.lds_sum, three words per event of the item (D', and the derivatives'
// sums).  The logarithms and ratios are formed after the last block, one thread per event.
template <int RINGS, int LEN, bool SOLO, int PITCH, bool VALUE>
__device__ __forceinline__ void loglik_item(const Geo& g, const Plan& p, const unsigned char* __restrict__ blocks,
                                            const BinItem it, const float* __restrict__ rho, double* __restrict__ Bimg,
                                            float* __restrict__ D_out, double* __restrict__ red,
                                            unsigned long long* __restrict__ cnt, const int32_t* __restrict__ order,
                                            unsigned char* smem, LogShared& ps) {
  constexpr int kEvents = SOLO ? 1 : 2, kHalf = WAVE / kEvents / 2;
  constexpr int kWords = (RINGS + 1) / 2;
  constexpr int kConst = ring_tails(kEvents, true);
  const int pitch = PITCH ? PITCH : p.pitch;
  const int npx = pitch * p.W;
  float* const rho_s = reinterpret_cast<float*>(smem + p.lds_img);
  double* const acc_s = reinterpret_cast<double*>(rho_s + npx);
  int* const off_s = reinterpret_cast<int*>(smem + p.lds_off);
  double* const D_s = reinterpret_cast<double*>(smem + p.lds_sum);
  float* const Du_s = reinterpret_cast<float*>(D_s + p.ev_per_wg);
  float* const Dw_s = Du_s + p.ev_per_wg;
  const int tid = threadIdx.x;
  const int lane = tid & (WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int waves = (int)(blockDim.x >> 6);
  const int nblk = (it.count + kEvents - 1) / kEvents;
  const unsigned char* const blk0 = blocks + (size_t)it.batch * (size_t)p.batch_bytes;
  unsigned char* const con_s = smem + wave * (2 * kConst);

  const int tz = it.bin % p.ntz;
  const int rest = it.bin / p.ntz;
  const int ty = rest % p.nty;
  const double tc = bin_slope(p, rest / p.nty);
  const int kmin = -max(shear_offset(g, tc, 0), shear_offset(g, tc, g.n_y - 1));
  const int rbase = ty * p.TY - p.HY;
  const int kbase = kmin + tz * p.TZ - p.HZ;
  LogGeo lg;
  lg.pix = uniform_f((float)g.pixel);
  lg.fa = uniform_f((float)g.fa);
  const double s2u = kHalfLog2e * 2.0 * g.u * g.pixel * g.pixel;  // (u in pixels, as the blocks have it rounded)
  lg.qlo = uniform_f((float)(s2u - (double)(float)s2u));

  uint32_t word[kWords];
  uint2 tails;
  auto fetch = [&](int q, int buf) {
    const unsigned char* blk = blk0 + (size_t)q * (size_t)p.batch_bytes;
    const int ln = fresh_lane();
    if (ln < kConst / 16)
      __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint4*>(blk + ln * 16), con_s + buf * kConst, 16, 0, 0);
#pragma unroll
    for (int j = 0; j < kWords; ++j)
      word[j] = reinterpret_cast<const uint32_t*>(blk + ring_words(kEvents, true))[j * WAVE + ln];
    tails = *reinterpret_cast<const uint2*>(blk + ring_tails(kEvents, true));
  };
  if (wave < nblk) fetch(wave, 0);
  if (tid == 0) ps.zero = ps.bad = 0u;
  if (tid < 3) ps.sum[tid] = 0.0;
  for (int r = tid; r < p.RY; r += blockDim.x) off_s[r] = shear_offset(g, tc, rbase + r);
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
      rho_s[q] = v;
      if constexpr (!VALUE) acc_s[q] = 0.0;
    }
  }
  __syncthreads();

  int buf = 0;
  for (int q = wave; q < nblk; q += waves, buf ^= 1) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this block's constants, words and tails have arrived
    const int ln = fresh_lane(), l = ln & (2 * kHalf - 1);
    const int lrow = l - kHalf, lstep = l < kHalf ? -kHalf : kHalf;
    const EvRow& c = reinterpret_cast<const EvRow*>(con_s + buf * kConst)[SOLO ? 0 : ln >> 5];
    const EvLog& cl = reinterpret_cast<const EvLog*>(con_s + buf * kConst + kEvents * sizeof(EvRow))[SOLO ? 0 : ln >> 5];
    const uint32_t t01 = __builtin_amdgcn_readfirstlane(tails.x), t23 = __builtin_amdgcn_readfirstlane(tails.y);
    uint32_t w[kWords];
#pragma unroll
    for (int j = 0; j < kWords; ++j) w[j] = word[j];
    if (q + waves < nblk) fetch(q + waves, buf ^ 1);

    auto tail = [&](int k) { return ((k < 2 ? t01 : t23) >> (16 * (k & 1))) & 0xffffu; };
    auto row = [&](int k, int H) { return ring_row(w[k >> 1] >> (16 * (k & 1)), c.mid + lrow + k * lstep, H); };
    auto event_sum = [&](float v) {  // over an event's lanes, to all of them
      if constexpr (SOLO) return wave_sum_dpp(v);
      const float h = half_sums_dpp(v);
      const float lo = lane_value(h, 31), hi = lane_value(h, 63);
      return ln < 32 ? lo : hi;
    };
    auto event_sum_d = [&](float v) {  // the same in double precision, for D'
      if constexpr (SOLO) return wave_sum_dpp_d((double)v);
      const double h = half_sums_dpp_d((double)v);
      const double lo = lane_value_d(h, 31), hi = lane_value_d(h, 63);
      return ln < 32 ? lo : hi;
    };
    // an event's sums (one lane each)
    auto finish = [&](double D, float Du, float Dw) {
      const int e = kEvents * q + (SOLO ? 0 : ln >> 5);
      if (l != 0 || e >= it.count) return;
      D_s[e] = D;
      if constexpr (!VALUE) {
        Du_s[e] = Du;
        Dw_s[e] = Dw;
      }
    };

    if ((t01 >> 14 & 3u) != kRowExact) {
      float D = 0.0f, Du = 0.0f, Dw = 0.0f;
      if constexpr (VALUE) {
        each_ring<0, RINGS>([&](auto kk) {
          constexpr int k = kk;
          const uint32_t tw = tail(k);
          const int wlh = (int)((tw & 127u) + 1) >> 1;
          const RingRow r = row(k, wlh);
          const float x = (float)(lrow + k * lstep);
          const RowF rk = ring_constants(c, x, r.kc + off_s[r.rl]);
          const float* const rr = rho_s + r.kc * pitch + r.rl;
          RowP rp;
          float F, S;
          if ((tw >> 14) == kRowPoly5) {
            F = row_poly<5>(rk, (float)r.nr - 0.5f, rp, lg.qlo);
            S = ring_value<5>(rp, rr, pitch, r.nl, r.nr, wlh);
          } else {
            F = row_poly<6>(rk, (float)r.nr - 0.5f, rp, lg.qlo);
            S = ring_value<6>(rp, rr, pitch, r.nl, r.nr, wlh);
          }
          if (r.nr > 0) D = fmaf(F, S, D);
        });
        const double De = event_sum_d(D);
        if (!__any(!(De < kFloatMax))) {
          finish(De, 0.0f, 0.0f);
          continue;
        }
      } else {
        RingCache<RINGS, LEN> cache;
        float F[RINGS];
        each_ring<0, RINGS>([&](auto kk) {
          constexpr int k = kk, H = ring_half_of(RINGS, LEN, k);
          const uint32_t tw = tail(k);
          const int wlh = (int)((tw & 127u) + 1) >> 1, wminh = (int)((tw >> 7) & 127u) >> 1;
          const RingRow r = row(k, H);
          const float x = (float)(lrow + k * lstep);
          const RowF rk = ring_constants(c, x, r.kc + off_s[r.rl]);
          const float* const rr = rho_s + (r.kc - H) * pitch + r.rl;
          RowP rp;
          float S0, X, G, Hs;
          if ((tw >> 14) == kRowPoly5) {
            Moments<5> M;
            F[k] = row_poly<5>(rk, (float)r.nr - 0.5f, rp, lg.qlo);
            ring_moments<H, 5>(rp, rr, pitch, r.nl, r.nr, wminh, wlh, cache.template ring<k>(), M);
            row_sums<5>(rk, M, X, G, Hs);
            S0 = M.m[0];
          } else {
            Moments<6> M;
            F[k] = row_poly<6>(rk, (float)r.nr - 0.5f, rp, lg.qlo);
            ring_moments<H, 6>(rp, rr, pitch, r.nl, r.nr, wminh, wlh, cache.template ring<k>(), M);
            row_sums<6>(rk, M, X, G, Hs);
            S0 = M.m[0];
          }
          float du, dw;
          row_derivatives(c, cl, x, lg, S0, X, G, Hs, du, dw);
          if (r.nr > 0) {
            D = fmaf(F[k], S0, D);
            Du = fmaf(F[k], du, Du);
            Dw = fmaf(F[k], dw, Dw);
          }
        });
        const double De = event_sum_d(D);
        Du = event_sum(Du);
        Dw = event_sum(Dw);
        if (!__any(!(De < kFloatMax && fabsf(Du) < kFloatMax && fabsf(Dw) < kFloatMax))) {
          finish(De, Du, Dw);
          const float invD = De > 0.0 ? (float)(1.0 / De) : 0.0f;
          each_ring<0, RINGS>([&](auto kk) {
            constexpr int k = kk, H = ring_half_of(RINGS, LEN, k);
            const uint32_t tw = tail(k);
            const int wlh = (int)((tw & 127u) + 1) >> 1, wminh = (int)((tw >> 7) & 127u) >> 1;
            const RingRow r = row(k, H);
            if (r.nr > 0 && invD > 0.0f)
              ring_back_f64<H>(cache.template ring<k>(), F[k] * invD, acc_s + (r.kc - H) * pitch + r.rl, pitch, r.nl,
                               r.nr, wminh, wlh);
          });
          continue;
        }
      }
    }

    // pixel by pixel, evaluated in both passes: rows that need it, and images so large that the sums without their
    // factor F, or the moments, overflow
    asm volatile("" ::: "memory");
    float D = 0.0f, Du = 0.0f, Dw = 0.0f;
    int nbad = 0, again = 0;
    const int first = opaque(0);
    for (int k = first; k < RINGS; ++k) {
      const RingRow r = row(k, 0);
      const float x = (float)(lrow + k * lstep), iS = 1.3862943611198906f;
      const RowF rk = ring_constants(c, x, r.kc + off_s[r.rl]);
      float S0 = 0.0f, X = 0.0f, G = 0.0f, H = 0.0f;
      for (int j = -r.nl; j < r.nr; ++j) {
        const float xj = (float)j + 0.5f;
        const float v = exact_at(rk, xj, &nbad) * rho_s[(r.kc + j) * pitch + r.rl];
        S0 += v;
        if constexpr (!VALUE) {
          if (v != 0.0f) {
            const float rq = __builtin_amdgcn_rsqf(fmaf(xj, rk.dkap, rk.kap0)), tg = fmaf(xj, rk.dgs, rk.gs0) * rq;
            const float gq = tg * rq;
            X = fmaf(v, fmaf(tg, tg, -fmaf(fmaf(rk.qa, xj, rk.qb), xj, rk.qc)), X);
            G = fmaf(v, gq, G);
            H = fmaf(v, fmaf(gq * gq, iS, rq * rq), H);
          }
        }
      }
      D += S0;
      if constexpr (!VALUE) {
        float du, dw;
        row_derivatives(c, cl, x, lg, S0, X, G, H, du, dw);
        if (r.nr > 0) {
          Du += du;
          Dw += dw;
        }
      }
    }
    if (nbad) atomicAdd(&ps.bad, (unsigned)nbad);
    const double De = event_sum_d(D);
    if constexpr (VALUE) {
      finish(De, 0.0f, 0.0f);
    } else {
      finish(De, event_sum(Du), event_sum(Dw));
      const float invD = De > 0.0 ? (float)(1.0 / De) : 0.0f;
      for (int k = first; k < RINGS; ++k) {
        const RingRow r = row(k, 0);
        const RowF rk = ring_constants(c, (float)(lrow + k * lstep), r.kc + off_s[r.rl]);
        for (int j = -r.nl; j < r.nr && invD > 0.0f; ++j)
          unsafeAtomicAdd(&acc_s[(r.kc + j) * pitch + r.rl], (double)(exact_at(rk, (float)j + 0.5f, &again) * invD));
      }
    }
  }
  __syncthreads();

  // the events' logarithms and ratios (see row_derivatives; b1^2 enters A by the blocks' rounded s2u)
  double a[3] = {0.0, 0.0, 0.0};
  const double cu = g.cu - 0.5 / g.u, iu = g.pixel * g.pixel / (double)(float)s2u, iw = 0.5 / (kHalfLog2e * g.w);
  unsigned zero = 0;
  for (int e = tid; e < it.count; e += (int)blockDim.x) {
    const double D = D_s[e];
    if (D > 0.0) {
      a[0] += log(D);
      if constexpr (!VALUE) {
        a[1] += cu + iu * ((double)Du_s[e] / D);
        a[2] += g.cw - iw * ((double)Dw_s[e] / D);
      }
    } else {
      ++zero;
    }
    if (D_out) D_out[order[it.start + e]] = D > 0.0 ? (float)(D * (double)(float)g.cnorm) : 0.0f;
  }
  if (zero) atomicAdd(&ps.zero, zero);
  for (int m = 0; m < (VALUE ? 1 : 3); ++m) {
    const double v = wave_sum_d(a[m]);
    if (lane == 0) unsafeAtomicAdd(&ps.sum[m], v);
  }
  // add the region's doubles to the global image (lanes along its rows, as in the pass on ring blocks)
  if constexpr (!VALUE) {
    const float inv_w = 1.0f / (float)p.W;
    for (int q = tid; q < p.RY * p.W; q += (int)blockDim.x) {
      const int rl = (int)(((float)q + 0.5f) * inv_w), cc = q - rl * p.W;
      const double v = acc_s[cc * pitch + rl];
      if (v == 0.0) continue;
      const int r = rbase + rl;
      const int k = kbase + cc + off_s[rl];
      if (r >= 0 && r < g.n_y && k >= 0 && k < g.n_z) unsafeAtomicAdd(&Bimg[(int64_t)r * g.n_z + k], v);
    }
  }
  __syncthreads();
  if (tid < (VALUE ? 1 : 3)) unsafeAtomicAdd(&red[tid], ps.sum[tid]);
  if (tid == 0) {
    if (ps.zero) atomicAdd(&cnt[C_ZERO_DEN], (unsigned long long)ps.zero);
    if (ps.bad) atomicAdd(&cnt[C_KAPPA_BAD], (unsigned long long)ps.bad);
  }
}

template <int SHAPE, int PITCH>
__global__ void __launch_bounds__((shape_threads(SHAPE, true)), (shape_waves_per_simd(SHAPE, true)))
    k_loglik_rings(Geo g, Plan p, const unsigned char* __restrict__ blocks, const BinItem* __restrict__ items,
                   const float* __restrict__ rho, double* __restrict__ B, float* __restrict__ D_out,
                   double* __restrict__ red, unsigned long long* __restrict__ cnt, const int32_t* __restrict__ order) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ LogShared ps;
  if ((unsigned long long)blockIdx.x >= cnt[C_ITEMS]) return;  // uniform over the workgroup
  loglik_item<shape_rings(SHAPE), shape_len(SHAPE), (SHAPE >= 1000), PITCH, false>(
      g, p, blocks, items[blockIdx.x], rho, B, D_out, red, cnt, order, smem, ps);
}

}  // namespace

template <int SHAPE>
hipError_t Rings<SHAPE>::loglik(const Geo& g, const Plan& p, const Workspace& ws, const float* rho, float* D_out,
                                hipStream_t st) {
  if (p.pitch != shape_pitch(SHAPE, 0) && p.pitch != shape_pitch(SHAPE, 1)) return hipErrorInvalidValue;
  auto kern = p.pitch == shape_pitch(SHAPE, 0) ? k_loglik_rings<SHAPE, shape_pitch(SHAPE, 0)>
                                               : k_loglik_rings<SHAPE, shape_pitch(SHAPE, 1)>;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kRingLdsLimit);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)p.max_items), dim3(64 * p.waves), p.lds_bytes, st, g, p, ws.batches,
                     ws.items, rho, ws.B, D_out, ws.red, ws.cnt, ws.order);
  return hipGetLastError();
}

}  // namespace jpet
