// Per-event preparation and spatial binning (iteration-invariant, run once per event list).
//
//   k_clear        counters and events per bin (and the accumulators, where asked for)
//   k_prepare      direct reconstruction (Eq. 2), ellipse rows (App. B, Sec. 3), validity; for the binned
//                  passes each event's bin and its rank in it, for the others the pixel count
//   k_scan         exclusive prefix sums over the bins of events, workgroup items and batch blocks; the items' order
//                  (k_scan_sums before it where there are many bins)
//   k_place        events in bin order, and the workgroup items: (bin, first event, count) with at most
//                  ev_per_wg events
//   k_build_rings, k_build_batches   the blocks the passes read, and the pixel count
#include <algorithm>

#include "jpet_rows.h"

namespace jpet {

namespace {

__device__ inline int clamp_index(double v, int lo, int hi) {
  if (!(v >= (double)lo)) return lo;   // also catches NaN
  if (v > (double)hi) return hi;
  return (int)v;
}

__device__ uint32_t bin_of(const Geo& g, const Plan& p, const EventRec& e) {
  int b = 0;
  if (p.ntb > 1) b = clamp_index(floor((e.t - p.tmin) / p.dt), 0, p.ntb - 1);
  const double tc = bin_slope(p, b);
  const int ic = clamp_index(rint((e.y - g.y0) * g.ipix), 0, g.n_y - 1);
  const int ty = ic / p.TY;
  const int kmin = -max(shear_offset(g, tc, 0), shear_offset(g, tc, g.n_y - 1));
  const double kz = (e.z - tc * e.y - g.z0) * g.ipix;
  const int tz = clamp_index(floor((kz - (double)kmin) / (double)p.TZ), 0, p.ntz - 1);
  return (uint32_t)(((int64_t)b * p.nty + ty) * p.ntz + tz);
}

// Direct reconstruction and rows of event j: the record with r1 < r0 for an invalid one.  The rows are those
// within the ellipse's half height, of which the outermost may hold no pixel centre; pixels (nullable):
// the ellipse's pixel count.
__device__ EventRec event_record(const Geo& g, const float* __restrict__ events, int64_t j, long long* pixels) {
  const float zu = events[3 * j], zd = events[3 * j + 1], dl = events[3 * j + 2];
  EventRec e;
  e.r0 = 0;
  e.r1 = -1;
  e.t = e.c = e.y = e.z = e.hs = 0.0;
  e.su = 1.0;
  const double hl = 0.5 * g.L;
  if (!(isfinite(zu) && isfinite(zd) && isfinite(dl) && fabs((double)zu) <= hl && fabs((double)zd) <= hl)) return e;
  // Eq. 2, first forms
  const double t = ((double)zu - (double)zd) / (2.0 * g.R);
  const double c = sqrt(1.0 + t * t);
  const double y = -0.5 * (double)dl / c;
  const double z = 0.5 * ((double)zu + (double)zd + 2.0 * y * t);
  e.t = t;
  e.c = c;
  e.y = y;
  e.z = z;
  // this event's sigma_z: sigma_z (1 + zedge zeta), zeta the mean of (z / (L/2))^2 over the
  // two hits (Sec. 3 after Eq. 12); u scales by the inverse square
  {
    const double xu = (double)zu / hl, xd = (double)zd / hl;
    const double f = 1.0 + g.zedge * (0.5 * (xu * xu + xd * xd));
    e.su = 1.0 / (f * f);
    e.hs = 0.5 / (g.um * e.su);
  }
  // rows within the ellipse's half height 1.5 sigma_dl / c (App. B)
  const double hy = 1.5 / (sqrt(g.wm) * c);
  double a = ceil((y - hy - g.y0) * g.ipix);
  double b = floor((y + hy - g.y0) * g.ipix);
  if (a < 0.0) a = 0.0;
  if (b > (double)(g.n_y - 1)) b = (double)(g.n_y - 1);
  if (!(a <= b)) return e;
  const int first = (int)a, last = (int)b;
  // valid when a pixel centre lies inside: the row nearest to the centre nearly always has one
  int klo, khi;
  bool some = row_interval(g, e, clamp_index(rint((y - g.y0) * g.ipix), first, last), &klo, &khi);
  if (pixels || !some) {
    long long count = 0;
    for (int i = first; i <= last; ++i)
      if (row_interval(g, e, i, &klo, &khi)) count += khi - klo + 1;
    some = count > 0;
    if (pixels) *pixels = count;
  }
  if (some) {
    e.r0 = first;
    e.r1 = last;
  }
  return e;
}

__global__ void k_clear(unsigned long long* __restrict__ cnt, uint32_t* __restrict__ bin_count, int64_t nbins,
                        unsigned long long* __restrict__ acc, int64_t npix) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < C_COUNT) cnt[i] = 0ull;
  if (i < nbins) bin_count[i] = 0u;
  if (i < npix) acc[i] = 0ull;
}

// Sums over the workgroup, added to the counters by one thread.
__device__ void add_counts(unsigned long long* __restrict__ cnt, unsigned long long valid, unsigned long long dropped,
                           unsigned long long pairs) {
  __shared__ unsigned long long s[3];
  if (threadIdx.x < 3) s[threadIdx.x] = 0ull;
  __syncthreads();
  valid = wave_sum_u64(valid);
  dropped = wave_sum_u64(dropped);
  pairs = wave_sum_u64(pairs);
  if ((threadIdx.x & (WAVE - 1)) == 0) {
    if (valid) atomicAdd(&s[0], valid);
    if (dropped) atomicAdd(&s[1], dropped);
    if (pairs) atomicAdd(&s[2], pairs);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    if (s[0]) atomicAdd(&cnt[C_VALID], s[0]);
    if (s[1]) atomicAdd(&cnt[C_DROPPED], s[1]);
    if (s[2]) atomicAdd(&cnt[C_PAIRS], s[2]);
  }
}

// Records for the passes without binning.
__global__ void __launch_bounds__(256) k_prepare_plain(Geo g, const float* __restrict__ events, int64_t n,
                                                       EventRec* __restrict__ ev,
                                                       unsigned long long* __restrict__ cnt) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  unsigned long long valid = 0, pairs = 0;
  if (j < n) {
    long long pixels = 0;
    const EventRec e = event_record(g, events, j, &pixels);
    ev[j] = e;
    valid = e.r1 >= e.r0;
    if (valid) pairs = (unsigned long long)pixels;
  }
  add_counts(cnt, valid, j < n ? 1 - valid : 0, pairs);
}

// Records, and each event's bin and rank in it.  A workgroup takes 1024 per events.  With LDS_RANK it counts
// them by bin in LDS first (nbins words) and adds each bin's count to the global one once: events
// crowd into few bins, and one global atomic per event puts most of them on a few addresses (10M
// events at 64 x 76 pixels: 2.7 ms for each of the former histogram and scatter).
template <bool LDS_RANK>
__global__ void __launch_bounds__(1024) k_prepare(Geo g, Plan p, const float* __restrict__ events, int64_t n, int per,
                                                  EventRec* __restrict__ ev, uint32_t* __restrict__ key,
                                                  uint32_t* __restrict__ rank, uint32_t* __restrict__ bin_count,
                                                  unsigned long long* __restrict__ cnt) {
  extern __shared__ uint32_t in_bin[];
  const int64_t j0 = (int64_t)blockIdx.x * 1024 * per + threadIdx.x;
  if constexpr (LDS_RANK) {
    for (int b = threadIdx.x; b < p.nbins; b += 1024) in_bin[b] = 0u;
    __syncthreads();
  }
  unsigned long long valid = 0, dropped = 0;
  for (int q = 0; q < per; ++q) {
    const int64_t j = j0 + 1024 * (int64_t)q;
    if (j >= n) break;
    const EventRec e = event_record(g, events, j, nullptr);
    ev[j] = e;
    uint32_t k = kNoBin;
    if (e.r1 >= e.r0) {
      ++valid;
      k = bin_of(g, p, e);
      rank[j] = atomicAdd(LDS_RANK ? &in_bin[k] : &bin_count[k], 1u);
    } else {
      ++dropped;
    }
    key[j] = k;
  }
  if constexpr (LDS_RANK) {
    __syncthreads();
    for (int b = threadIdx.x; b < p.nbins; b += 1024)
      if (const uint32_t c = in_bin[b]) in_bin[b] = atomicAdd(&bin_count[b], c);
    __syncthreads();
    for (int q = 0; q < per; ++q) {  // this thread's own events
      const int64_t j = j0 + 1024 * (int64_t)q;
      if (j >= n) break;
      if (key[j] != kNoBin) rank[j] += in_bin[key[j]];
    }
  }
  add_counts(cnt, valid, dropped, 0ull);
}

// Exclusive prefix sums over the bins.  The full items of all bins come first, then the bins' rests, those in
// the largest eighth of their range first: the pass's workgroups are dispatched in this order, so the shortest
// ones fill the chip's last round.  Against rests in the order of the bins, the pass over 375,000 events on
// 256^2 takes 252 us instead of 295, over 100,000 on 400^2 115 instead of 125, over 10M there 5.98 ms
// instead of 6.16.  Latency bounds the scan: every block of 1024 bins sums the bins before its own for itself,
// out of L2, where one block with 100 bins per thread took 155 us for 103,000 of them.  That is quadratic in the
// bins, so above kScanBins of them the blocks, at most kScanBlocks of them, read sums that k_scan_sums has formed
// of each block's bins (the whole preparation of 20,000 events on 1024^2: 46,440 bins 146 us either way, 185,760
// 248 -> 148, 3.06M 14,330 -> 357; of 100,000 events on 4096^2, 6.6M bins: 64.7 -> 0.63 ms).
constexpr int kScanBins = 1 << 16, kScanBlocks = 2048;
constexpr int kRestClasses = 8;
__device__ inline int rest_class(uint32_t rest, int ev_per_wg) {  // 0: the largest; rest in [1, ev_per_wg)
  return kRestClasses - 1 - (int)(rest * (uint32_t)kRestClasses / (uint32_t)ev_per_wg);
}

// What a bin adds to the sums: its events, full items and batches, and its rest's class (-1: no rest).
constexpr int kScanOwn = 3, kScanPer = kScanOwn + kRestClasses;
struct BinSums {
  uint32_t own[kScanOwn];
  int cls;
  __device__ BinSums(uint32_t c, int ev_per_wg, int ev_per_batch)
      : own{c, c / ev_per_wg, (c + ev_per_batch - 1) / ev_per_batch},
        cls(c % ev_per_wg ? rest_class(c % ev_per_wg, ev_per_wg) : -1) {}
};

// The sums of each block's bins (chunks of 1024), kScanPer words a block.
__global__ void __launch_bounds__(1024) k_scan_sums(int nbins, int chunks, int ev_per_wg, int ev_per_batch,
                                                    const uint32_t* __restrict__ bin_count, uint32_t* __restrict__ sums) {
  __shared__ uint32_t part[kScanPer];
  if (threadIdx.x < kScanPer) part[threadIdx.x] = 0u;
  __syncthreads();
  uint32_t v[kScanPer] = {};
  for (int ch = 0; ch < chunks; ++ch) {
    const int64_t b = ((int64_t)blockIdx.x * chunks + ch) * 1024 + threadIdx.x;
    const BinSums s(b < nbins ? bin_count[b] : 0u, ev_per_wg, ev_per_batch);
    for (int q = 0; q < kScanOwn; ++q) v[q] += s.own[q];
#pragma unroll
    for (int q = 0; q < kRestClasses; ++q) v[kScanOwn + q] += s.cls == q ? 1u : 0u;
  }
#pragma unroll
  for (int q = 0; q < kScanPer; ++q) {
    for (int off = WAVE / 2; off > 0; off >>= 1) v[q] += __shfl_down(v[q], off);
    if ((threadIdx.x & (WAVE - 1)) == 0 && v[q]) atomicAdd(&part[q], v[q]);
  }
  __syncthreads();
  if (threadIdx.x < kScanPer) sums[(int64_t)blockIdx.x * kScanPer + threadIdx.x] = part[threadIdx.x];
}

// sums: k_scan_sums's, or null for blocks of one chunk that sum the bins themselves.
__global__ void __launch_bounds__(1024) k_scan(int nbins, int chunks, int ev_per_wg, int ev_per_batch,
                                               const uint32_t* __restrict__ bin_count, const uint32_t* __restrict__ sums,
                                               uint32_t* __restrict__ bin_start, uint32_t* __restrict__ item_start,
                                               uint32_t* __restrict__ rest_start, uint32_t* __restrict__ batch_start,
                                               unsigned long long* __restrict__ cnt) {
  constexpr int kBefore = kScanOwn, kAll = kScanPer, kSums = kAll + 1 + kRestClasses;
  // events, full items, batches and the classes' rests of the bins before this block's; full items and the
  // classes' rests of all bins
  __shared__ uint32_t part[kSums][1024 / WAVE], base[kSums];
  const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
  const int64_t first = (int64_t)blockIdx.x * chunks * 1024;
  uint32_t v[kSums] = {};
  if (sums) {
    for (int k = threadIdx.x; k < (int)gridDim.x; k += 1024) {
      const uint32_t before = k < (int)blockIdx.x ? 1u : 0u;
      for (int q = 0; q < kScanPer; ++q) {
        const uint32_t x = sums[(int64_t)k * kScanPer + q];
        v[q] += before * x;
        if (q == 1) v[kAll] += x;
        if (q >= kBefore) v[kAll + 1 + q - kBefore] += x;
      }
    }
  } else {
    for (int b = threadIdx.x; b < nbins; b += 1024) {
      const BinSums s(bin_count[b], ev_per_wg, ev_per_batch);
      const uint32_t before = b < first ? 1u : 0u;
      for (int q = 0; q < kBefore; ++q) v[q] += before * s.own[q];
      v[kAll] += s.own[1];
#pragma unroll
      for (int q = 0; q < kRestClasses; ++q) {
        const uint32_t one = s.cls == q ? 1u : 0u;
        v[kBefore + q] += before * one;
        v[kAll + 1 + q] += one;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < kSums; ++q) {
    for (int off = WAVE / 2; off > 0; off >>= 1) v[q] += __shfl_down(v[q], off);
    if (lane == 0) part[q][wave] = v[q];
  }
  __syncthreads();
  if (threadIdx.x < kSums) {
    uint32_t sum = 0;
    for (int w = 0; w < 1024 / WAVE; ++w) sum += part[threadIdx.x][w];
    base[threadIdx.x] = sum;
  }
  __syncthreads();
  // this block's own bins, a chunk at a time: sums over the wavefront's lanes, then over the wavefronts before
  for (int ch = 0; ch < chunks; ++ch) {
    const int64_t b = first + (int64_t)ch * 1024 + threadIdx.x;
    const BinSums s(b < nbins ? bin_count[b] : 0u, ev_per_wg, ev_per_batch);
    uint32_t run[kBefore], rank = 0;
#pragma unroll
    for (int q = 0; q < kBefore; ++q) {
      run[q] = s.own[q];
      for (int off = 1; off < WAVE; off <<= 1) {
        const uint32_t up = __shfl_up(run[q], off);
        if (lane >= off) run[q] += up;
      }
      if (lane == WAVE - 1) part[q][wave] = run[q];
      run[q] -= s.own[q];
    }
#pragma unroll
    for (int q = 0; q < kRestClasses; ++q) {
      const unsigned long long in = __ballot(s.cls == q);
      if (s.cls == q) rank = (uint32_t)__popcll(in & ((1ull << lane) - 1ull));
      if (lane == 0) part[kBefore + q][wave] = (uint32_t)__popcll(in);
    }
    __syncthreads();
    for (int q = 0; q < kBefore; ++q) {
      run[q] += base[q];
      for (int w = 0; w < wave; ++w) run[q] += part[q][w];
    }
    if (s.cls >= 0) {
      rank += base[kAll] + base[kBefore + s.cls];
      for (int q = 0; q < s.cls; ++q) rank += base[kAll + 1 + q];
      for (int w = 0; w < wave; ++w) rank += part[kBefore + s.cls][w];
    }
    if (b < nbins) {
      bin_start[b] = run[0];
      item_start[b] = run[1];
      batch_start[b] = run[2];
      rest_start[b] = rank;
    }
    if (b == nbins - 1) {
      bin_start[nbins] = run[0] + s.own[0];
      uint32_t items = base[kAll];
      for (int q = 0; q < kRestClasses; ++q) items += base[kAll + 1 + q];
      cnt[C_ITEMS] = items;
    }
    __syncthreads();
    if (threadIdx.x < kScanPer)
      for (int w = 0; w < 1024 / WAVE; ++w) base[threadIdx.x] += part[threadIdx.x][w];
    __syncthreads();
  }
}

// Thread j places event j; thread b writes bin b's items.
__global__ void __launch_bounds__(256) k_place(const uint32_t* __restrict__ key, const uint32_t* __restrict__ rank,
                                               int64_t n, int nbins, int ev_per_wg, int ev_per_batch,
                                               const uint32_t* __restrict__ bin_count,
                                               const uint32_t* __restrict__ bin_start,
                                               const uint32_t* __restrict__ item_start,
                                               const uint32_t* __restrict__ rest_start,
                                               const uint32_t* __restrict__ batch_start, int32_t* __restrict__ order,
                                               BinItem* __restrict__ items) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j < n && key[j] != kNoBin) order[bin_start[key[j]] + rank[j]] = (int32_t)j;
  if (j >= nbins) return;
  const int b = (int)j;
  const uint32_t c = bin_count[b], full = c / (uint32_t)ev_per_wg;
  for (uint32_t i = 0; i * ev_per_wg < c; ++i) {
    const uint32_t s = i * ev_per_wg;
    BinItem it;
    it.bin = b;
    it.start = (int32_t)(bin_start[b] + s);
    it.count = (int32_t)min((uint32_t)ev_per_wg, c - s);
    it.batch = (int32_t)(batch_start[b] + s / ev_per_batch);
    items[i < full ? item_start[b] + i : rest_start[b]] = it;
  }
}

// The per-event constants of the binned MLEM pass (EvRow) for a bin whose region starts at pixel
// row rbase and (sheared) column kbase, in double precision.  With r the region row, the row's
// y is Y = Yb + pix r and dy = Y - y~ = pix r - yr, both linear in r; each row constant of the
// kernel (Eq. 7-12; see EvRow) is then a polynomial of degree <= 2 in r, expanded here.  unit: the length b1 is
// measured in (1 mm, or the pixel for ring blocks).
__device__ EvRow event_row_constants(const Geo& g, const EventRec& e, int index, int rbase, int kbase, double unit) {
  const double pix = g.pixel, t = e.t, c = e.c, c2 = c * c, f = g.fa;
  const double u = g.u * e.su, w = g.w;  // u: this event's sigma_z^-2
  const double Yb = g.y0 + (double)rbase * pix;
  const double yr = e.y - Yb;                          // dy = pix r - yr
  const double zr = e.z - (g.z0 + (double)kbase * pix);
  const double rs = 0.84932180028801904272;            // sqrt(log2(e) / 2)
  const double S = kHalfLog2e;
  // kappa without its b1 term: A1 (R^2 + Y^2) + A2 Y^2 + A3 Y dy + GK (fa Y + 2 dy)
  const double A1 = 2.0 * u * c2 * c2, A2 = w * f * f * c2 * t * t, A3 = 4.0 * w * c2 * (1.0 + 2.0 * t * t);
  const double GK = -4.0 * g.gamma * g.R * c2 * c * t;
  const double KB = -4.0 * u * t * c2;                 // kappa's slope in b1 per unit Y
  // sqrt(S) gamma^ without its b1 term: rs (G1 Y dy + GG dy); its slope in b1 per unit Y: rs GB
  const double G1 = 2.0 * f * w * c2 * t, GG = -4.0 * g.gamma * g.R * c2 * c, GB = -2.0 * u * c2;
  const double Q3 = S * 4.0 * w * c2;                  // S q = S 2u b1^2 + Q3 dy^2
  EvRow k;
  k.B0 = (float)((t * yr - zr) / unit);
  k.BT = (float)(-t * pix / unit);
  // Y^2 = Yb^2 + 2 Yb pix r + pix^2 r^2,  Y dy = -Yb yr + (Yb - yr) pix r + pix^2 r^2
  k.K0 = (float)(A1 * g.R * g.R + (A1 + A2) * Yb * Yb - A3 * Yb * yr + GK * (f * Yb - 2.0 * yr));
  k.K1 = (float)(((A1 + A2) * 2.0 * Yb + A3 * (Yb - yr) + GK * (f + 2.0)) * pix);
  k.K2 = (float)((A1 + A2 + A3) * pix * pix);
  k.KB0 = (float)(KB * Yb * unit);
  k.KB1 = (float)(KB * pix * unit);
  k.S0 = (float)(rs * (-G1 * Yb * yr - GG * yr));
  k.S1 = (float)(rs * (G1 * (Yb - yr) + GG) * pix);
  k.S2 = (float)(rs * G1 * pix * pix);
  k.GB0 = (float)(rs * GB * Yb * unit);
  k.GB1 = (float)(rs * GB * pix * unit);
  k.Q0 = (float)(Q3 * yr * yr);
  k.Q1 = (float)(-2.0 * Q3 * yr * pix);
  k.Q2 = (float)(Q3 * pix * pix);
  const double s2u = S * 2.0 * u;
  k.qa = (float)(s2u * pix * pix);
  k.QB = (float)(2.0 * s2u * pix);
  k.s2u = (float)(s2u * unit * unit);
  k.index = index;
  k.mid = 0;
  return k;
}

// The pixel row nearest to an event's point (it may lie outside the grid).
__device__ inline int centre_row(const Geo& g, const EventRec& e) {
  return (int)floor((e.y - g.y0) * g.ipix + 0.5);
}

// How the pass on ring blocks may evaluate a row of nl + nr pixels about its centre, k its constants there.
// kappa is affine along the row: unless it keeps a margin of 1e-3 of its central value at both ends, the
// pixels need the kappa <= 0 test (kRowExact).  Otherwise the exponent of the kernel is expanded about
// the centre in y = delta x (the pass's RowP, with the same names): the remainder after x^5 is at most
// (w x^2 y^4 + log2(e)/2 y^6 / 6) / (1 - y), beside log2(e)/2 (y^4 / 12 + 2 y^5 / 15) for the
// logarithm's last two terms (taken as -delta times the one before), that after the economised x^7 and x^8 at
// most w x^2 (y^5 / 64 + y^6 / 128 + y^7 / (1 - y)) + log2(e)/2 (y^7 / 448 + y^8 / 1024 + y^9 / (9 (1 - y))),
// at the row's end.  The polynomial is taken while that stays below 1e-7 in the exponent (base 2), under
// the rounding of S q, and while no slot of the register cache (the first H pixels from the centre),
// pixels past the row's ends included, can overflow.  Where the line lies: with strips at 450 mm nearly all
// rows take x^5, of the paper's setting (R = 130 mm, sigma_z = 10 mm) half need x^6, few the exact form.
__device__ inline int row_mode(const RowF& k, int nl, int nr, int H) {
  const float L = (float)kHalfLog2e, M = (float)nr, X = (float)(H + 1);
  const float klo = fmaf(-(float)nl, k.dkap, k.kap0), khi = fmaf((float)nr, k.dkap, k.kap0);
  if (!(k.kap0 > 0.0f && fminf(klo, khi) > 1e-3f * k.kap0)) return kRowExact;
  const float rq = __builtin_amdgcn_rsqf(k.kap0), dl = k.dkap * rq * rq, y = fabsf(dl) * M;
  const float h0 = k.gs0 * rq, h1 = k.dgs * rq, d = h1 - dl * h0, w = d * d;
  // the exponent at any slot
  const float z = fabsf(dl) * X, c1 = h0 * (h1 + d) - L * dl - k.qb, c2 = w + 0.5f * L * dl * dl - k.qa;
  const float most = fabsf(c1) * X + fmaxf(c2, 0.0f) * X * X + 2.0f * (w * X * X + L) * z * (1.0f + z * (1.0f + z * (1.0f + z)));
  if (!(most < 100.0f) || !(y < 0.25f)) return kRowExact;
  const float wm = w * M * M, y2 = y * y, y4 = y2 * y2, q = __builtin_amdgcn_rcpf(1.0f - y);
  if ((wm * y4 + L * y4 * y2 / 6.0f) * q + L * y4 * (1.0f / 12.0f + 2.0f / 15.0f * y) < 1e-7f) return kRowPoly5;
  const float y5 = y4 * y, y6 = y4 * y2, y7 = y6 * y;
  if (wm * (y5 / 64.0f + y6 / 128.0f + y7 * q) + L * (y7 / 448.0f + y4 * y4 / 1024.0f + y7 * y2 * q / 9.0f) < 1e-7f)
    return kRowPoly6;
  return kRowExact;
}

// Batch blocks of the binned pass: one workgroup per item builds, for each batch of ev_per_batch
// events, the per-event constants and the thread words.  A thread owns one row segment of at most
// the register cache's length: every ellipse row has a first segment, and when the plan splits
// rows (p.segs = 2) each row longer than the cache also has a second one, its remaining pixels.
// The segments of one level of one event form a "group" of consecutive rows.  Rows are given to
// threads so that a wavefront holds rows of nearly equal length: each group's rows are cut into
// rings of 32 rows around its central row (ring 0: the 32 central rows; ring k: 16 rows above and
// 16 below ring k-1) and a remainder at its two tips.  Half-wavefront slots take the rings ordered
// by ring index, then by group, so a wavefront pairs two rings at the same distance from their
// ellipses' centres; the tips of all groups fill the remaining threads.  Within a half-wavefront
// the rows are consecutive, so its LDS accesses fall into distinct banks (the two halves of a
// wavefront can still meet in a bank).
constexpr int kBuildBatch = 32;
constexpr int kBuildGroups = 2 * kBuildBatch;
constexpr int kBuildSlots = 64;

__global__ void __launch_bounds__(1024) k_build_batches(Geo g, Plan p, const EventRec* __restrict__ ev,
                                                        const int32_t* __restrict__ order,
                                                        const BinItem* __restrict__ items,
                                                        unsigned char* __restrict__ blocks,
                                                        unsigned long long* __restrict__ cnt) {
  __shared__ EventRec ev_s[kBuildBatch];
  // groups: g < nb is event g's first segments over all its rows; nb + g its second segments,
  // over the rows from its first to its last row longer than the register cache (none: 0 rows)
  __shared__ int grp_r0[kBuildGroups], grp_n[kBuildGroups];
  __shared__ int K_s[kBuildGroups], top_s[kBuildGroups];
  __shared__ unsigned char slot_g[kBuildSlots], slot_k[kBuildSlots];
  __shared__ int tip_cum[kBuildGroups + 1];
  __shared__ int nslots_s;
  __shared__ unsigned outside_s;
  if ((unsigned long long)blockIdx.x >= cnt[C_ITEMS]) return;
  const BinItem it = items[blockIdx.x];
  const int tz = it.bin % p.ntz;
  const int rest = it.bin / p.ntz;
  const int ty = rest % p.nty;
  const int tb = rest / p.nty;
  const double tc = bin_slope(p, tb);
  const int kmin = -max(shear_offset(g, tc, 0), shear_offset(g, tc, g.n_y - 1));
  const int rbase = ty * p.TY - p.HY;
  const int kbase = kmin + tz * p.TZ - p.HZ;
  const int tid = threadIdx.x;
  const int lane = tid & (WAVE - 1);
  if (tid == 0) outside_s = 0u;
  unsigned long long pairs = 0;  // pixels of the rows this thread builds
  for (int e0 = 0, bi = 0; e0 < it.count; e0 += p.ev_per_batch, ++bi) {
    const int nb = min(p.ev_per_batch, it.count - e0);
    const int ng = p.segs > 1 ? 2 * nb : nb;
    unsigned char* blk = blocks + (size_t)(it.batch + bi) * (size_t)p.batch_bytes;
    uint32_t* words = reinterpret_cast<uint32_t*>(blk + p.cbytes);
    __syncthreads();
    if (tid < nb) {
      const int j = order[it.start + e0 + tid];
      const EventRec e = ev[j];
      ev_s[tid] = e;
      grp_r0[tid] = 0;
      grp_n[tid] = e.r1 - e.r0 + 1;
      if (p.segs > 1) {  // the rows longer than the register cache
        int first = -1, last = -2;
        for (int i = e.r0; i <= e.r1; ++i) {
          int klo, khi;
          if (row_interval(g, e, i, &klo, &khi) && khi - klo + 1 > p.maxlen) {
            if (first < 0) first = i - e.r0;
            last = i - e.r0;
          }
        }
        grp_r0[nb + tid] = first < 0 ? 0 : first;
        grp_n[nb + tid] = last - first + 1 > 0 ? last - first + 1 : 0;
      }
      if (p.loglik) {
        const float t = (float)e.t, c2 = (float)(e.c * e.c), u = (float)(g.u * e.su), w = (float)g.w,
                    fa = (float)g.fa;
        EvConst k;
        k.yr = (float)(e.y - (g.y0 + (double)rbase * g.pixel));
        k.zr = (float)(e.z - (g.z0 + (double)kbase * g.pixel));
        k.index = j;
        k.S2u = (float)(kHalfLog2e * 2.0 * (g.u * e.su));
        k.t = t;
        k.A1 = 2.0f * u * c2 * c2;
        k.A2 = w * fa * fa * c2 * t * t;
        k.A3 = 4.0f * w * c2 * (1.0f + 2.0f * t * t);
        k.KB = -4.0f * u * t * c2;
        k.G1 = 2.0f * fa * w * c2 * t;
        k.GB = -2.0f * u * c2;
        k.Q3s = (float)kHalfLog2e * 4.0f * w * c2;
        {
          const double c3 = e.c * e.c * e.c;
          k.GK = (float)(-4.0 * g.gamma * g.R * c3 * e.t);
          k.GG = (float)(-4.0 * g.gamma * g.R * c3);
        }
        k.pad[0] = k.pad[1] = 0;
        reinterpret_cast<EvConst*>(blk)[tid] = k;
      } else {
        reinterpret_cast<EvRow*>(blk)[tid] = event_row_constants(g, e, j, rbase, kbase, 1.0);
      }
    }
    __syncthreads();
    if (tid < WAVE) {  // ring slots (ring-major, then group) and the tip prefix
      const int nrows = tid < ng ? grp_n[tid] : 0;
      const int mrow = nrows >> 1;
      const int K = min(mrow, nrows - mrow) >> 4;
      const int T = nrows - 32 * K;
      if (tid < ng) {
        K_s[tid] = K;
        top_s[tid] = mrow - 16 * K;
      }
      const int Kmax = wave_max_i(K);
      int base_slot = 0;
      for (int k = 0; k < Kmax; ++k) {
        const unsigned long long msk = __ballot(K > k);
        const int before = __popcll(msk & ((1ull << lane) - 1ull));
        if (K > k) {
          slot_g[base_slot + before] = (unsigned char)tid;
          slot_k[base_slot + before] = (unsigned char)k;
        }
        base_slot += __popcll(msk);
      }
      int incl = T;
#pragma unroll
      for (int off = 1; off < WAVE; off <<= 1) {
        const int o = __shfl_up(incl, off, WAVE);
        if (lane >= off) incl += o;
      }
      if (tid < ng) tip_cum[tid] = incl - T;
      if (tid == ng - 1) tip_cum[ng] = incl;
      if (tid == 0) nslots_s = base_slot;
    }
    __syncthreads();
    const int nslots = nslots_s;
    int gi = -1, ri = 0;  // group and row within the group
    if (tid < 32 * nslots) {
      const int sl = tid >> 5, l = tid & 31;
      gi = slot_g[sl];
      const int k = slot_k[sl];
      const int mrow = grp_n[gi] >> 1;
      ri = k == 0 ? mrow - 16 + l : (l < 16 ? mrow - 16 * (k + 1) + l : mrow + 16 * k + (l - 16));
    } else if (tid - 32 * nslots < tip_cum[ng]) {
      const int q = tid - 32 * nslots;
      int lo = 0, hi = ng - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (tip_cum[mid] <= q) lo = mid; else hi = mid - 1;
      }
      gi = lo;
      const int qq = q - tip_cum[gi];
      const int top = top_s[gi];
      ri = qq < top ? qq : (grp_n[gi] >> 1) + 16 * K_s[gi] + (qq - top);
    }
    uint32_t word = 0u;
    bool guard = false;  // this segment may reach kappa <= 0: the pass tests every pixel
    if (gi >= 0) {
      const int e = gi < nb ? gi : gi - nb;
      const EventRec er = ev_s[e];
      const int i = er.r0 + grp_r0[gi] + ri;
      int klo, khi;
      if (row_interval(g, er, i, &klo, &khi)) {
        int n = khi - klo + 1;
        if (gi < nb) {  // first segment
          pairs += n;
          if (n > p.maxlen && p.segs > 1) n = p.maxlen;
        } else {        // second segment: the pixels past the first
          klo += p.maxlen;
          n -= p.maxlen;
        }
        if (n > 0) {
          const int rl = i - rbase;
          const int kl = klo - shear_offset(g, tc, i) - kbase;
          if (rl < 0 || rl >= p.RY || kl < 0 || kl + n > p.W || n > p.maxlen) {
            atomicAdd(&outside_s, 1u);
          } else {
            word = ((uint32_t)kl << kWordCol) | ((uint32_t)rl << kWordRow) | ((uint32_t)n << kWordLen) |
                   ((uint32_t)e << kWordEv);
            // kappa is affine along the row: its smallest value is at one of the segment's two
            // ends; segments whose ends both keep a margin of 1e-3 of the first value can skip
            // the test
            double kf, ks;
            (void)row_constants(g, er, i, klo, &kf, &ks);
            const double kend = kf + (double)(n - 1) * ks;
            guard = !(kf > 1e-3 * fabs(kf) && kend > 1e-3 * fabs(kf));
          }
        }
      }
    }
    if (tid < 64 * p.waves) {
      words[tid] = word;
      const int len = (int)((word >> kWordLen) & 127u);
      const int wl = wave_max_i(len);
      const int wmin = -wave_max_i(len > 0 ? -len : -wl);  // shortest non-empty row (0: none)
      const bool wguard = __any(guard);
      // does each half-wavefront hold rows of one event only (the pass then reduces the
      // denominators per half, without the per-event loop)?
      const int ev = (int)((word >> kWordEv) & 31u);
      const unsigned long long act = __ballot(len > 0);
      const unsigned long long half = lane < 32 ? 0xffffffffull : 0xffffffff00000000ull;
      const unsigned long long mine = act & half;
      const int lead = mine ? __ffsll((long long)mine) - 1 : (lane & 32);
      const int ev_lead = __shfl(ev, lead, WAVE);
      const bool split = __any(len > 0 && ev != ev_lead);
      // (a half with no rows takes the other half's event)
      int ev_lo = __shfl(ev_lead, 0, WAVE), ev_hi = __shfl(ev_lead, 32, WAVE);
      if (!(act & 0xffffffffull)) ev_lo = ev_hi;
      if (!(act >> 32)) ev_hi = ev_lo;
      if (lane == 0) {
        words[64 * p.waves + (tid >> 6)] = (uint32_t)wl | (wguard ? kRowExact << kModeShift : 0u);
        words[65 * p.waves + (tid >> 6)] =
            (uint32_t)wmin |
            (split ? 0u : (1u << kHalfBit) | ((uint32_t)ev_lo << kHalfLo) | ((uint32_t)ev_hi << kHalfHi));
      }
    }
  }
  __syncthreads();
  if (tid == 0 && outside_s) atomicAdd(&cnt[C_OUTSIDE], (unsigned long long)outside_s);
  add_counts(cnt, 0ull, 0ull, pairs);
}

// The largest of each 16-bit half over the wavefront (all lanes active), to every lane.
__device__ __forceinline__ uint32_t wave_max_u16x2(uint32_t v) {
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  auto step = [](uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
  };
  v = step(v, __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, true));   // quad_perm [1,0,3,2]
  v = step(v, __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, true));   // quad_perm [2,3,0,1]
  v = step(v, __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, true));  // row_half_mirror
  v = step(v, __builtin_amdgcn_update_dpp(0, v, 0x140, 0xf, 0xf, true));  // row_mirror
  v = step(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, true));  // row_bcast:15 into rows 1 and 3
  v = step(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, true));  // row_bcast:31 into rows 2 and 3
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// An event for the rows of its ring block, in pixels from its central row and the column nearest to its point.
struct RowsOf {
  float fy, zf;        // its point: rows past the central row, columns past kcen
  float A, hs;         // 4 wm c^2 and hs in pixels
  float t;
  int32_t kcen;
  int16_t r0, r1;      // its rows, from the central row on (r1 < r0: no event)
  int16_t mid, mode;   // the central row in the region; how all its rows may be evaluated, kRowExact: row by row
};
static_assert(sizeof(RowsOf) == 32, "RowsOf is read in 16-byte units");

__device__ RowsOf rows_of(const Geo& g, const EventRec& e, int mid, bool none) {
  RowsOf o;
  const double yp = (e.y - g.y0) * g.ipix, zp = (e.z - g.z0) * g.ipix, kc = rint(zp);
  o.fy = (float)(yp - (double)mid);
  o.zf = (float)(zp - kc);
  o.A = (float)(4.0 * g.wm * e.c * e.c * g.pixel * g.pixel);
  o.hs = (float)(e.hs * g.ipix * g.ipix);
  o.t = (float)e.t;
  o.kcen = (int)kc;
  o.r0 = (int16_t)(none ? 0 : e.r0 - mid);
  o.r1 = (int16_t)(none ? -1 : e.r1 - mid);
  o.mid = 0;
  o.mode = (int16_t)kRowExact;
  return o;
}

// row_interval in single precision, for row x from the central row on.  False when the result is not
// certain: an end within 5e-4 of a pixel centre, or a row within 0.01 of the ellipse's top in
// 9 - 4 wm c^2 dy^2.  (Rounding: dy^2 and the product lose at most 4e-6 of 9, so a half chord of up to 32
// pixels 2e-4 where 0.01 is left under the root; the centre's column, at most 150 away, 5e-5.)
__device__ __forceinline__ bool row_interval_fast(const RowsOf& e, int x, int n_z, int* klo, int* khi) {
  const float dy = (float)x - e.fy;
  const float rem = fmaf(-e.A * dy, dy, 9.0f);
  const float H = __builtin_amdgcn_sqrtf(fmaxf(rem, 0.0f) * e.hs);
  const float c = fmaf(e.t, dy, e.zf), a = c - H, b = c + H;
  const float lo = ceilf(a), hi = floorf(b);
  *klo = max(e.kcen + (int)lo, 0);
  *khi = rem > 0.0f ? min(e.kcen + (int)hi, n_z - 1) : -1;
  const float near = fminf(fminf(lo - a, 1.0f - (lo - a)), fminf(b - hi, 1.0f - (b - hi)));
  return rem < -0.01f || (rem > 0.01f && near > 5e-4f);
}

// row_mode for all rows of an event (half height X rows, at most 2 H pixels long) at once: over each of
// eight bands of rows with the largest value that each of its terms has there.  kRowExact: not decided
// by these bounds.
__device__ inline int all_rows_mode(const EvRow& c, float X, int H) {
  int mode = (int)kRowPoly5;
  const float h = 0.125f * X;
  for (int s = 0; s < 8; ++s) {
    const float x = ((float)s - 3.5f) * 0.25f * X, out = (fabsf(x) - h) / X;  // band centre, its inner edge
    const int M = min(H, (int)(sqrtf(1.0f - out * out) * (float)H) + 1);
    const float kb = fabsf(fmaf(c.KB1, x, c.KB0)) + fabsf(c.KB1) * h, gb = fabsf(fmaf(c.GB1, x, c.GB0)) + fabsf(c.GB1) * h;
    const float b1 = (float)(M + 1);  // of a row's centre, rows cut by the grid's edge included
    RowF k;
    k.kap0 = fmaf(fmaf(c.K2, x, c.K1), x, c.K0) - fmaf(fabsf(c.K2), h, fabsf(fmaf(2.0f * c.K2, x, c.K1))) * h - kb * b1;
    k.dkap = kb;
    // (signs that add up in w and in the slope)
    k.gs0 = -(fabsf(fmaf(fmaf(c.S2, x, c.S1), x, c.S0)) + fmaf(fabsf(c.S2), h, fabsf(fmaf(2.0f * c.S2, x, c.S1))) * h +
              gb * b1);
    k.dgs = gb;
    k.qa = c.s2u;
    k.qb = 2.0f * c.s2u * b1;
    k.qc = 0.0f;
    mode = max(mode, row_mode(k, M, M, H));
  }
  return mode;
}

// Ring blocks (plans with rings): one workgroup per item, first the row constants of its events, one
// per thread, then one wavefront per block, one lane per row of its event and ring.
__global__ void __launch_bounds__(256, 6) k_build_rings(Geo g, Plan p, const EventRec* __restrict__ ev,
                                                     const int32_t* __restrict__ order,
                                                     const BinItem* __restrict__ items,
                                                     unsigned char* __restrict__ blocks,
                                                     unsigned long long* __restrict__ cnt) {
  extern __shared__ __align__(16) unsigned char smem[];  // the events' RowsOf, the column shift of every region row
  if ((unsigned long long)blockIdx.x >= cnt[C_ITEMS]) return;
  const BinItem it = items[blockIdx.x];
  const int tz = it.bin % p.ntz;
  const int rest = it.bin / p.ntz;
  const int ty = rest % p.nty;
  const double tc = bin_slope(p, rest / p.nty);
  const int kmin = -max(shear_offset(g, tc, 0), shear_offset(g, tc, g.n_y - 1));
  const int rbase = ty * p.TY - p.HY;
  const int kbase = kmin + tz * p.TZ - p.HZ;
  const int epb = p.ev_per_batch, lpe = WAVE / epb;  // events per block, lanes per event
  const int tid = threadIdx.x, lane = tid & (WAVE - 1), l = lane & (lpe - 1);
  const int nblk = (it.count + epb - 1) / epb;
  unsigned char* const blk0 = blocks + (size_t)it.batch * (size_t)p.batch_bytes;
  RowsOf* const rows_s = reinterpret_cast<RowsOf*>(smem);
  int* const off_s = reinterpret_cast<int*>(rows_s + p.ev_per_wg + 1);
  for (int r = tid; r < p.RY; r += blockDim.x) off_s[r] = shear_offset(g, tc, rbase + r) + kbase;
  for (int e = tid; e < nblk * epb; e += blockDim.x) {
    const int j = order[it.start + min(e, it.count - 1)];
    const EventRec er = ev[j];
    // polynomials in the rows from the event's central row on: the rounding of their coefficients
    // then stays below that of the rows' own values
    const int mid = centre_row(g, er);
    EvRow k = event_row_constants(g, er, e < it.count ? j : -1, mid, kbase, g.pixel);  // (-1: no event)
    k.mid = mid - rbase;
    reinterpret_cast<EvRow*>(blk0 + (size_t)(e / epb) * (size_t)p.batch_bytes)[e % epb] = k;
    if (p.loglik) {
      const double w = g.w, c2 = er.c * er.c, t2 = er.t * er.t;
      EvLog q;
      q.A2 = (float)(w * g.fa * g.fa * c2 * t2);
      q.A3 = (float)(4.0 * w * c2 * (1.0 + 2.0 * t2));
      q.GG = (float)(-4.0 * g.gamma * g.R * c2 * er.c);
      q.GK = (float)(-4.0 * g.gamma * g.R * c2 * er.c * er.t);
      const double Y0 = g.y0 + (double)mid * g.pixel;
      q.Y0 = (float)Y0;
      q.yr = (float)(er.y - Y0);
      q.pad[0] = q.pad[1] = 0.0f;
      reinterpret_cast<EvLog*>(blk0 + (size_t)(e / epb) * (size_t)p.batch_bytes + epb * sizeof(EvRow))[e % epb] = q;
    }
    RowsOf o = rows_of(g, er, mid, e >= it.count);
    o.mid = (int16_t)k.mid;
    o.mode = (int16_t)all_rows_mode(k, (float)p.HY, p.ring_half[0]);
    rows_s[e] = o;
  }
  __syncthreads();
  int outside = 0;
  unsigned long long pairs = 0;
  for (int q = tid >> 6; q < nblk; q += blockDim.x >> 6) {
    unsigned char* const blk = blk0 + (size_t)q * (size_t)p.batch_bytes;
    const int e = epb * q + lane / lpe;
    const RowsOf er = rows_s[e];
    const int mid = er.mid + rbase;
    uint32_t tails[4] = {0, 0, 0, 0}, word = 0;
    int mode = 0;
    for (int k = 0; k < p.rings; ++k) {
      const int x = l - lpe / 2 + k * (l < lpe / 2 ? -lpe / 2 : lpe / 2), i = mid + x;
      int klo = 0, khi = -1, n = 0, kl = 0, m = (int)kRowPoly5;
      if (x >= er.r0 && x <= er.r1 && !row_interval_fast(er, x, g.n_z, &klo, &khi) &&
          !row_interval(g, ev[order[it.start + e]], i, &klo, &khi))
        khi = klo - 1;
      if (khi >= klo) {
        n = khi - klo + 1;
        pairs += n;
        const int rl = i - rbase;
        kl = rl >= 0 && rl < p.RY ? klo - off_s[rl] : -1;
        if (kl < 0 || kl + n > p.W || n > 2 * p.ring_half[k]) {
          ++outside;
          n = 0;
        }
      }
      const int nl = n >> 1, nr = n - nl, kc = kl + nl;
      const uint32_t ends = wave_max_u16x2(n > 0 ? (uint32_t)n | (uint32_t)(128 - n) << 16 : 0u);
      const int wl = (int)(ends & 0xffffu), wmin = wl ? 128 - (int)(ends >> 16) : 0;
      if (n > 0) {
        m = er.mode;
        if (m == (int)kRowExact) {
          const EvRow& c = reinterpret_cast<const EvRow*>(blk)[lane / lpe];
          m = row_mode(ring_constants(c, (float)x, kc + off_s[i - rbase] - kbase), nl, nr, p.ring_half[k]);
        }
        // the chunks of two pairs the pass runs for this ring, from the row's centre, stay in the region and
        // its slack
        const int reach = min(p.ring_half[k], (((wl + 1) >> 1) + 1) & ~1);
        if (kc - reach < -p.slack || kc + reach > p.W + p.slack) m = (int)kRowExact;
      }
      m = __any(m == (int)kRowExact) ? (int)kRowExact : __any(m == (int)kRowPoly6) ? (int)kRowPoly6 : (int)kRowPoly5;
      mode = max(mode, m);
      tails[k] = (uint32_t)wl | ((uint32_t)wmin << 7) | ((uint32_t)m << 14);
      word |= (n > 0 ? (uint32_t)kl | ((uint32_t)n << 8) : 0u) << (16 * (k & 1));
      if ((k & 1) || k + 1 == p.rings) {
        reinterpret_cast<uint32_t*>(blk + ring_words(epb, p.loglik))[(k >> 1) * WAVE + lane] = word;
        word = 0;
      }
    }
    if (mode == (int)kRowExact)  // one row of a block that needs the exact form: all take it
      for (int k = 0; k < 4; ++k) tails[k] = (tails[k] & 0x3fffu) | (kRowExact << 14);
    if (lane == 0)
      *reinterpret_cast<uint2*>(blk + ring_tails(epb, p.loglik)) =
          make_uint2(tails[0] | tails[1] << 16, tails[2] | tails[3] << 16);
  }
  outside = (int)wave_sum_u64((unsigned long long)outside);
  if (lane == 0 && outside) atomicAdd(&cnt[C_OUTSIDE], (unsigned long long)outside);
  add_counts(cnt, 0ull, 0ull, pairs);
}

int blocks_for(int64_t n, int block) { return (int)((n + block - 1) / block); }

}  // namespace

hipError_t launch_prepare(const Geo& g, const Plan& p, const float* events, int64_t n, const Workspace& ws,
                          hipStream_t st) {
  const int64_t nb = p.tiled ? p.nbins : 0;
  const int64_t clear = std::max<int64_t>(C_COUNT, std::max(nb, ws.clear_acc));
  hipLaunchKernelGGL(k_clear, dim3(blocks_for(clear, 256)), dim3(256), 0, st, ws.cnt, ws.bin_count, nb, ws.acc,
                     ws.clear_acc);
  if (!p.tiled) {
    if (n > 0)
      hipLaunchKernelGGL(k_prepare_plain, dim3(blocks_for(n, 256)), dim3(256), 0, st, g, events, n, ws.ev, ws.cnt);
    return hipGetLastError();
  }
  if (n > 0) {
    // events per thread: one while that leaves compute units idle, up to 32 (the more, the fewer bins a
    // workgroup's events have to themselves); counting in LDS while its bins fit and are fewer than 8
    // per event (else the counts are few, and clearing and adding them costs more)
    const int per = (int)std::min<int64_t>(32, std::max<int64_t>(1, n / (1024 * 256)));
    const size_t lds = sizeof(uint32_t) * (size_t)nb;
    if (lds <= (size_t)kPrepareLdsLimit && nb <= 8 * 1024 * per) {
      const hipError_t e = hipFuncSetAttribute((const void*)k_prepare<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                               kPrepareLdsLimit);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(k_prepare<true>, dim3(blocks_for(n, 1024 * per)), dim3(1024), lds, st, g, p, events, n, per,
                         ws.ev, ws.key, ws.rank, ws.bin_count, ws.cnt);
    } else {
      hipLaunchKernelGGL(k_prepare<false>, dim3(blocks_for(n, 1024 * per)), dim3(1024), 0, st, g, p, events, n, per,
                         ws.ev, ws.key, ws.rank, ws.bin_count, ws.cnt);
    }
  }
  // (the sums of many bins lie in ws.B, which only the log-likelihood's pass uses, cleared before; an image too small
  // for them, of very wide strips, leaves the blocks to sum the bins)
  const bool many = nb > kScanBins && (int64_t)g.n_y * g.n_z * (int64_t)sizeof(double) >=
                                          (int64_t)sizeof(uint32_t) * kScanPer * kScanBlocks;
  uint32_t* const sums = many ? reinterpret_cast<uint32_t*>(ws.B) : nullptr;
  const int chunks = many ? blocks_for(nb, 1024 * kScanBlocks) : 1, scan = blocks_for(nb, 1024 * chunks);
  if (many)
    hipLaunchKernelGGL(k_scan_sums, dim3(scan), dim3(1024), 0, st, p.nbins, chunks, p.ev_per_wg, p.ev_per_batch,
                       ws.bin_count, sums);
  hipLaunchKernelGGL(k_scan, dim3(scan), dim3(1024), 0, st, p.nbins, chunks, p.ev_per_wg, p.ev_per_batch, ws.bin_count,
                     sums, ws.bin_start, ws.item_start, ws.rest_start, ws.batch_start, ws.cnt);
  if (n <= 0) return hipGetLastError();
  hipLaunchKernelGGL(k_place, dim3(blocks_for(n > nb ? n : nb, 256)), dim3(256), 0, st, ws.key, ws.rank, n, p.nbins,
                     p.ev_per_wg, p.ev_per_batch, ws.bin_count, ws.bin_start, ws.item_start, ws.rest_start,
                     ws.batch_start, ws.order, ws.items);
  if (p.rings) {
    hipLaunchKernelGGL(k_build_rings, dim3((unsigned)p.max_items), dim3(256),
                       sizeof(RowsOf) * (size_t)(p.ev_per_wg + 1) + sizeof(int) * (size_t)p.RY, st, g, p,
                       ws.ev, ws.order, ws.items, ws.batches, ws.cnt);
  } else {
    hipLaunchKernelGGL(k_build_batches, dim3((unsigned)p.max_items), dim3(64 * p.waves), 0, st, g, p, ws.ev, ws.order,
                       ws.items, ws.batches, ws.cnt);
  }
  return hipGetLastError();
}

}  // namespace jpet
