// The kernel of Eq. 7-12 along one pixel row, exactly and as the exponential of a polynomial.
#pragma once

#include "jpet_device.h"

namespace jpet {

namespace {

// Single-precision kernel constants along one pixel row (Eq. 7-12) as functions of the pixel's offset
// x in the row, from its first pixel (jpet_binned.h) or from its centre (jpet_rings.h):
//   kappa = kap0 + x dkap,  sqrt(S) gamma = gs0 + x dgs,  S q = (qa x + qb) x + qc
// (qa = S 2u pixel^2 depends on the event through its sigma_z)
// and P / (sqrt(det C^-1) / 2 pi) = kappa^-1/2 exp2(S gamma^2 / kappa - S q), S = log2(e) / 2.
// The off-diagonal gamma of C^-1 enters only kappa and gamma^ through per-row constants: with
// b1 = b2, the gamma terms of b C^-1 b cancel (so the ellipse does not depend on gamma) while
// kappa gains -4 gamma R c^3 t (fa y + 2 dy) and gamma^ gains -4 gamma R c^3 dy.
struct RowF {
  float kap0, dkap, gs0, dgs, qa, qb, qc;
};

// The constants at the centre of a row of a ring block: x the row from its event's central row on, col
// the first pixel right of the centre (region-local column plus the row's shift).  b1 is in pixels, so that one
// rounded constant, s2u, stands for u in every term of S q.
__device__ __forceinline__ RowF ring_constants(const EvRow& c, float x, int col) {
  const float b1 = ((float)col - 0.5f) + fmaf(c.BT, x, c.B0);
  const float kb = fmaf(c.KB1, x, c.KB0), gb = fmaf(c.GB1, x, c.GB0);
  const float sb = c.s2u * b1;
  RowF k;
  k.kap0 = fmaf(kb, b1, fmaf(fmaf(c.K2, x, c.K1), x, c.K0));
  k.dkap = kb;
  k.gs0 = fmaf(gb, b1, fmaf(fmaf(c.S2, x, c.S1), x, c.S0));
  k.dgs = gb;
  k.qa = c.s2u;
  k.qb = sb + sb;
  k.qc = fmaf(sb, b1, fmaf(fmaf(c.Q2, x, c.Q1), x, c.Q0));
  return k;
}

// The same row as F exp2(E(x)), E a polynomial without constant term.  With kappa_0, gs_0 at the
// centre, delta = dkap / kappa_0, h0 = gs_0 kappa_0^-1/2, h1 = dgs kappa_0^-1/2 and
// w = (h1 - delta h0)^2 the exponent is exactly
//   h0^2 - S q(0) - log2(kappa_0)/2 + (h0 (2 h1 - delta h0) - qb) x - qa x^2
//     + w x^2 / (1 + delta x) - log2(1 + delta x) / 2,
// and delta x, the relative change of kappa along the row, is at most a few percent: the last two
// terms are expanded, to x^5 (kRowPoly5) or x^6 with the x^7 and x^8 terms economised onto the lower ones
// (Chebyshev; kRowPoly6).  row_mode() keeps only rows whose remainder is below 1e-7 in E, less than
// the rounding of S q itself; the others, and rows that may reach kappa <= 0, take the exact form.
// Per pixel this costs 3 (3.5) FMAs and v_exp_f32 in place of 9 FMAs or multiplies, v_rsq_f32 and
// v_exp_f32: the pixels x = i + 1/2 and x = -(i + 1/2) share the even part and the odd part's
// factor, and every power of x is a literal.
struct RowP {
  float c1, c2, c3, c4, c5, c6;
};

constexpr float kHalfLog2eF = 0.72134752044448170368f;

// A register-cache entry that pass 2 does not read: any value, set by no instruction (keeping the
// previous batch's value would keep the whole cache live through pass 1).
__device__ __forceinline__ float unread() { return __builtin_nondeterministic_value(0.0f); }

// The polynomial form of a row; half: the largest |x| of its pixels; qlo: what qa has lost by its rounding, the same
// for all rows (the log-likelihood's derivatives sum over many events what is left of terms that cancel).
// Returns F.
template <int DEG>
__device__ __forceinline__ float row_poly(const RowF& k, float half, RowP& p, float qlo = 0.0f) {
  const float rq = __builtin_amdgcn_rsqf(k.kap0);
  const float dl = k.dkap * (rq * rq);
  const float h0 = k.gs0 * rq, h1 = k.dgs * rq;
  const float d = fmaf(-dl, h0, h1), w = d * d, dl2 = dl * dl;
  p.c1 = fmaf(h0, h1 + d, -fmaf(kHalfLog2eF, dl, k.qb));
  p.c2 = fmaf(0.5f * kHalfLog2eF, dl2, (w - qlo) - k.qa);
  p.c3 = -dl * fmaf(kHalfLog2eF / 3.0f, dl2, w);
  if constexpr (DEG == 5) {  // the logarithm's x^4 and x^5 terms only nearly, within row_mode's bound
    p.c4 = -dl * p.c3;
    p.c5 = -dl * p.c4;
  } else {
    p.c4 = dl2 * fmaf(kHalfLog2eF / 4.0f, dl2, w);
    p.c5 = -dl * dl2 * fmaf(kHalfLog2eF / 5.0f, dl2, w);
    const float dl4 = dl2 * dl2, m2 = half * half;
    p.c6 = dl4 * fmaf(kHalfLog2eF / 6.0f, dl2, w);
    const float c7 = -dl * dl4 * fmaf(kHalfLog2eF / 7.0f, dl2, w) * m2;
    const float c8 = dl4 * dl2 * fmaf(kHalfLog2eF / 8.0f, dl2, w) * m2;
    p.c6 = fmaf(2.0f, c8, p.c6);
    p.c5 = fmaf(1.75f, c7, p.c5);
    p.c4 = fmaf(-1.25f * m2, c8, p.c4);
    p.c3 = fmaf(-0.875f * m2, c7, p.c3);
    p.c2 = fmaf(0.25f * m2 * m2, c8, p.c2);
    p.c1 = fmaf(0.109375f * m2 * m2, c7, p.c1);
  }
  return rq * __builtin_amdgcn_exp2f(fmaf(h0, h0, -k.qc));
}

// exp2(E) at x = -(i + 1/2) (lo) and x = i + 1/2 (hi).
template <int DEG>
__device__ __forceinline__ void poly_pair(const RowP& p, int i, float& lo, float& hi) {
  const float x = (float)i + 0.5f, X = x * x;
  float ev = fmaf(p.c4, X, p.c2);
  if constexpr (DEG == 6) ev = fmaf(fmaf(p.c6, X, p.c4), X, p.c2);
  ev *= X;
  const float od = fmaf(fmaf(p.c5, X, p.c3), X, p.c1);
  lo = __builtin_amdgcn_exp2f(fmaf(od, -x, ev));
  hi = __builtin_amdgcn_exp2f(fmaf(od, x, ev));
}

}  // namespace

}  // namespace jpet
