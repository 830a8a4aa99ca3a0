// The CV sums of the first-order (triangular) shape in double (Sec. II.B, Eq.
// cv_def with T_h and its two-fold convolution; the shape in dev_tri.hpp).
//
// Both terms are piecewise polynomials of the separation D. The unit of
// length here is a cell, L / C, and s = 1 / (the half-width in cells). With
// u = D s, 6 B(u) / 8 is
//   (4 - 6 u^2 + 3 u^3) / 8 - (u - 1)^3_+ / 2 + (u - 2)^3_+ / 8
// and max(0, 1 - u) is 1 - u + (u - 1)_+; the spline's periodic image is (D -
// (C - 2 / s))^3_+ s^3 / 8. Particles are sorted into C cells, and an ordered
// pair whose cells differ by e (mod C) has D = e + v - u with u, v the offsets
// within the cells. A polynomial of D therefore sums over a whole band of
// cell pairs through
//   Q_m(e) = sum over the band's pairs of (v - u)^m,  m = 0..3,
// which follow from the cells' centred moments sum (u - 1/2)^k and do not
// depend on the width. A band that ends before the knot p1 = h takes the inner
// polynomial (and 1 - u), one that ends before p2 = 2h the outer one, (2 -
// u)^3 / 8; none reaches past 2h. A band that holds a knot adds, per particle,
// the powers (p1 - D)^3 and (p1 - D), or (p2 - D)^3, of the partners before it:
// those ahead of it in one sorted cell and those of at most one whole cell,
// from the moments of the cell's prefixes. So a partner outside the support
// enters no sum, a sum without partners is exactly 0, and none is negative.
// (The image's power (D - p2)^3 is taken likewise beyond its knot, C - 2h.)
// Pairs within a cell (D has a kink at 0) give sum |v - u|^m the same way. So a
// width costs a binary search and two cubics per particle and C / 2 cubics,
// against every pair within its support (29 % of n^2 / 2 on average over a list up
// to half the period).
// Widths narrower than a cell walk each particle's partners within the support
// (they follow it in the sorted array) pair by pair: there the moments would
// lose the figures that the separation has. Offsets are exact (C is a power of two,
// the sorted values are positions in cell units) and s <= 1 elsewhere, so the
// sums are as accurate as the direct ones (5.1e-16 against 8.4e-16 of the
// pair kernel at 30,001 particles and 32 widths, against direct sums).
//
// Kernels: cell counts (global integer atomics), scatter (each workgroup
// scans the counts for itself), rank within the cell (the order the atomics
// gave is replaced by the order of the values, so that every sum below has a
// fixed order), prefix moments, the knots' terms, band sums, and per width
// the cubics, the partial sums and the objective. What bounds it is launches
// and latency: at 30,001 particles and 32 widths the scan takes 54 us (1600 us
// over the pairs), 20 us of it the knots' terms (chains of dependent loads),
// the rest seven kernels of 2 to 8 us. A sample within a few cells pays for its
// ranks and, at widths narrower than a cell, for its pairs: 30,001 within 1e-4 L
// 1.6 ms over 32 widths from L / 1024 (4.8 over the pairs), from L / 16384, six of
// them narrower than a cell, 6.1 (4.8).
#include <algorithm>
#include <cmath>

#include "dev_layout.hpp"
#include "dev_fourier.hpp"
#include "kde_internal.hpp"

namespace kde {

namespace {

constexpr int kTriMinCells = 8, kTriMaxCells = 2048;  // 4 moments of 2048 cells: 64 KB of LDS
constexpr int64_t kTriMany = int64_t(1) << 26;        // particles from which the knots' terms take kTriPer per thread
constexpr int kTriPer = 4;
constexpr int kBandBlock = 256;
constexpr int kBands = kBandBlock / 64;                 // bands per workgroup, one per wave

// About 16 particles per cell up to the limit, fewer for small samples: ranking
// within a cell costs its count per particle, the band sums C^2 / 2
// products. Up to 2048 particles 8 to 16 per cell, so that what the cells take
// fits the pair layout's workspace (carve_tri).
int tri_cells(int64_t n) {
  int c = 256;
  while (c < kTriMaxCells && int64_t(c) * 16 < n) c *= 2;
  while (c > kTriMinCells && int64_t(c) * 8 >= n) c /= 2;
  return c;
}

struct TriWidths {
  int B, C, emax;           // bands 1..emax are needed by the widest support
  double L;
  double h[KDE_MAX_KAPPAS];
};

// A width in cell units: s = 1 / p1, its knots p1 and p2 (2 p1, or past half
// the period its image's, folded).
struct TriKnots {
  double s, p1, p2;
  bool image;   // h > L / 4: the spline reaches its periodic image
  bool direct;  // narrower than a cell: pair by pair
  bool half;    // a knot in the last band (e = C / 2), which also holds its mirror image: that band pair by pair
};

__device__ __forceinline__ TriKnots tri_knots(double h, double L, int C) {
  TriKnots k;
  const double g = h / L;
  k.p1 = g * double(C);
  k.p2 = 2.0 * k.p1;
  k.s = 1.0 / k.p1;
  k.image = g > 0.25;
  if (k.p2 > 0.5 * double(C)) k.p2 = fmax(double(C) - k.p2, 0.0);
  k.direct = k.p1 < 1.0;
  k.half = fmax(k.p1, k.p2) > double(C / 2 - 1);
  return k;
}
// Position in cell units, in [0, C) (NaN for a non-finite one), and its cell.
__device__ __forceinline__ double cell_position(double x, double L, int C) {
  double z = (wrap_d(x, L) / L) * double(C);
  if (z >= double(C) || z < 0.0) z = 0.0;  // rounded to the period's end
  return z;
}
__device__ __forceinline__ int cell_index(double z) { return int(z); }  // 0 for NaN

__global__ void __launch_bounds__(kBlock) tri_zero_kernel(int* __restrict__ count, int C, unsigned int* done) {
  const int c = blockIdx.x * kBlock + threadIdx.x;
  if (c < C) count[c] = 0;
  if (c == 0) *done = 0u;
}

__global__ void __launch_bounds__(kBlock) tri_count_kernel(const double* __restrict__ x, int64_t n, double L, int C,
                                                          int* __restrict__ count, int* __restrict__ rank,
                                                          uint32_t* status) {
  const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (i >= n) return;
  const double xv = x[i];
  note_numeric(status, !isfinite(xv), false);
  rank[i] = atomicAdd(&count[cell_index(cell_position(xv, L, C))], 1);
}

// Exclusive prefix of the counts by every workgroup for itself (the first
// writes it out), then its particles to their cells.
__global__ void __launch_bounds__(kBlock) tri_scatter_kernel(const double* __restrict__ x, int64_t n, double L, int C,
                                                            const int* __restrict__ count,
                                                            const int* __restrict__ rank, int* __restrict__ start,
                                                            double* __restrict__ cells) {
  __shared__ int base[kTriMaxCells];
  __shared__ int tot[kBlock / 64];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int64_t i = int64_t(blockIdx.x) * kBlock + t;
  const double z = i < n ? cell_position(x[i], L, C) : 0.0;
  const int r = i < n ? rank[i] : 0;
  for (int c = t; c < C; c += kBlock) base[c] = count[c];
  __syncthreads();
  const int per = C > kBlock ? C / kBlock : 1;
  const int cells_of = t * per < C ? per : 0;
  int own = 0;
  for (int k = 0; k < cells_of; ++k) own += base[t * per + k];
  int incl = own;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int y = __shfl_up(incl, d, 64);
    if (lane >= d) incl += y;
  }
  if (lane == 63) tot[w] = incl;
  __syncthreads();
  int run = incl - own;
  for (int k = 0; k < w; ++k) run += tot[k];
  for (int k = 0; k < cells_of; ++k) {
    const int v = base[t * per + k];
    base[t * per + k] = run;
    run += v;
  }
  __syncthreads();
  if (blockIdx.x == 0) {
    for (int c = t; c < C; c += kBlock) start[c] = base[c];
    if (t == 0) start[C] = int(n);
  }
  if (i < n) cells[base[cell_index(z)] + r] = z;
}

// The order within each cell: a value's rank is the number of smaller ones
// (compared as integers: positions are >= 0, and a NaN counts as largest;
// equal values keep the places they have, which changes nothing).
__global__ void __launch_bounds__(kBlock) tri_rank_kernel(const double* __restrict__ cells, int64_t n,
                                                         const int* __restrict__ start, double* __restrict__ sorted) {
  const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (i >= n) return;
  const double z = cells[i];
  const int c = cell_index(z);
  const int lo = start[c], hi = start[c + 1];
  const uint64_t key = uint64_t(__double_as_longlong(z));
  int r = 0;
#pragma unroll 8
  for (int j = lo; j < hi; ++j) {
    const uint64_t k = uint64_t(__double_as_longlong(cells[j]));
    r += (k < key || (k == key && j < int(i))) ? 1 : 0;
  }
  sorted[lo + r] = z;
}

// K workgroup sums in a fixed order (wave butterflies, then the waves).
template <int K, int W>
__device__ __forceinline__ void sums_of_block(double (&v)[K], double (*red)[K]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = wave_sum(v[k]);
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) red[w][k] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) {
    v[k] = 0.0;
#pragma unroll
    for (int q = 0; q < W; ++q) v[k] += red[q][k];
  }
  __syncthreads();
}

// Moments sum 1, d, d^2, d^3 of offsets from a cell's middle.
struct __align__(16) Mom4 {
  double m0, m1, m2, m3;
};
__device__ __forceinline__ Mom4 operator-(const Mom4& a, const Mom4& b) {
  return Mom4{a.m0 - b.m0, a.m1 - b.m1, a.m2 - b.m2, a.m3 - b.m3};
}
// sum (d - t), sum (d - t)^2, sum (d - t)^3.
__device__ __forceinline__ double shift1(const Mom4& m, double t) { return fma(-t, m.m0, m.m1); }
__device__ __forceinline__ double shift2(const Mom4& m, double t) { return fma(t, fma(t, m.m0, -2.0 * m.m1), m.m2); }
__device__ __forceinline__ double shift3(const Mom4& m, double t) {
  return fma(t, fma(t, fma(-t, m.m0, 3.0 * m.m1), -3.0 * m.m2), m.m3);
}

struct Mom3 {
  double m1, m2, m3;
};
// Adds a particle at offset d.
__device__ __forceinline__ void mom_add(Mom3& m, double d) {
  const double d2 = d * d;
  m.m1 += d;
  m.m2 += d2;
  m.m3 = fma(d2, d, m.m3);
}

// Wave per cell: the moments of the particles before each even place of the
// sorted array in its cell (pre[place / 2], without the count, which the places
// give), and of the whole cell (mu). A lane takes two places, and the lanes'
// sums meet in a shuffle scan: one load and one scan per 128 particles, where a
// thread per cell waits for each of its particles in turn (15,000 in one cell: ms).
__global__ void __launch_bounds__(kBlock) tri_prefix_kernel(const double* __restrict__ z,
                                                           const int* __restrict__ start, int C,
                                                           Mom3* __restrict__ pre, Mom4* __restrict__ mu) {
  const int lane = threadIdx.x & 63, c = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  if (c >= C) return;
  const double mid = double(c) + 0.5;
  const int lo = start[c], hi = start[c + 1];
  Mom3 carry{0.0, 0.0, 0.0};
  for (int base = lo & ~1; base < hi; base += 128) {
    const int e = base + 2 * lane;
    Mom3 m{0.0, 0.0, 0.0};
    if (e >= lo && e < hi) mom_add(m, z[e] - mid);
    if (e + 1 < hi) mom_add(m, z[e + 1] - mid);
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const Mom3 o{__shfl_up(m.m1, d, 64), __shfl_up(m.m2, d, 64), __shfl_up(m.m3, d, 64)};
      if (lane >= d) m = Mom3{o.m1 + m.m1, o.m2 + m.m2, o.m3 + m.m3};
    }
    Mom3 b{__shfl_up(m.m1, 1, 64), __shfl_up(m.m2, 1, 64), __shfl_up(m.m3, 1, 64)};
    if (lane == 0) b = Mom3{0.0, 0.0, 0.0};
    if (e >= lo && e < hi) pre[e >> 1] = Mom3{carry.m1 + b.m1, carry.m2 + b.m2, carry.m3 + b.m3};
    carry.m1 += __shfl(m.m1, 63, 64);
    carry.m2 += __shfl(m.m2, 63, 64);
    carry.m3 += __shfl(m.m3, 63, 64);
  }
  if (lane == 0) mu[c] = Mom4{double(hi - lo), carry.m1, carry.m2, carry.m3};
}
// The moments of the particles [lo, a) of the cell that starts at lo, whose
// middle is mid, for a place lo < a of the cell (elsewhere a value that means
// nothing). Its loads are made at once and stay in the arrays.
struct Prefixes {
  const double* z;
  const Mom3* pre;
  int last;  // n - 1
  __device__ __forceinline__ Mom4 of(int a, int lo, double mid) const {
    a = min(a, last);
    Mom3 m = pre[a >> 1];
    const double before = z[max(a - 1, 0)];
    mom_add(m, (a & 1) ? before - mid : 0.0);
    return Mom4{double(a - lo), m.m1, m.m2, m.m3};
  }
};

// Where a knot p of particle i falls: in cell J = I + rel (mod C), at t from
// the cell's start; [a, b) narrows to the first particle at or beyond it.
struct KnotPlace {
  int f, rel, J, a, b, lo, hi;
  double base, t;
};
__device__ __forceinline__ KnotPlace knot_place(double ui, int I, double p, int C, const int* __restrict__ start) {
  KnotPlace k;
  k.f = int(p);
  k.t = ui + (p - double(k.f));
  k.rel = k.t >= 1.0 ? k.f + 1 : k.f;
  if (k.rel > k.f) k.t -= 1.0;
  k.J = (I + k.rel) & (C - 1);
  k.base = double(k.J);
  k.a = k.lo = start[k.J];
  k.b = k.hi = start[k.J + 1];
  return k;
}
// Sums of (p - D) and (p - D)^3 over the partners before the knot in the bands
// that hold it (e <= last): those ahead of it in its own cell, and all of the
// cell of the band before (`prev`, that of band f). Each is a sum of positive
// terms, so what rounding leaves below 0 is 0.
__device__ __forceinline__ void before_knot(const KnotPlace& k, int last, const Mom4& own, const Mom4& prev,
                                            const Prefixes& pre, double& s1, double& s3) {
  s1 = s3 = 0.0;
  if (k.rel <= last && k.a > k.lo) {
    const Mom4 m = k.a < k.hi ? pre.of(k.a, k.lo, k.base + 0.5) : own;
    s1 = fmax(0.0, -shift1(m, k.t - 0.5));
    s3 = fmax(0.0, -shift3(m, k.t - 0.5));
  }
  if (k.rel > k.f && k.f <= last) {
    s1 += fmax(0.0, -shift1(prev, k.t + 0.5));
    s3 += fmax(0.0, -shift3(prev, k.t + 0.5));
  }
}
// The sum of (D - p)^3 over those beyond it: the rest of its own cell, and the
// next band's whole cell.
__device__ __forceinline__ double beyond_knot(const KnotPlace& k, bool between, int last, const Mom4& own,
                                              const Mom4& next, const Prefixes& pre) {
  double s3 = 0.0;
  if (k.rel <= last && k.a < k.hi) 
    s3 = fmax(0.0, shift3(k.a > k.lo ? own - pre.of(k.a, k.lo, k.base + 0.5) : own, k.t - 0.5));
  if (k.rel == k.f && between && k.f + 1 <= last) s3 += fmax(0.0, shift3(next, k.t - 1.5));
  return s3;
}

// Slot y of the grid: y < B, width y's terms at its knots (or all of its
// pairs); y = B, sum |v - u|^m over the pairs within cells. P = 1 particle per
// thread (two or four: 24 and 33 us against 20), kTriPer where there are so many
// that their partial sums would need more room. A slot's partial sums go to
// part[(y gridDim.x + x) 2 ..], four of them for y = B. A non-finite position makes
// every sum NaN.
template <int P>
__global__ void __launch_bounds__(kBlock) tri_knots_kernel(const double* __restrict__ z, int64_t n,
                                                          const int* __restrict__ start,
                                                          const Mom3* __restrict__ pre_of,
                                                          const Mom4* __restrict__ mu, TriWidths W, double* __restrict__ part) {
  __shared__ double red[kBlock / 64][4];
  const Prefixes pre{z, pre_of, int(n - 1)};
  const int C = W.C, slot = W.B - int(blockIdx.y);  // the widest widths, the longest (but for the narrowest), start first
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  const int64_t first = int64_t(blockIdx.x) * (P * kBlock) + threadIdx.x;
  if (slot == W.B) {
    for (int64_t i = first, q = 0; q < P && i < n; ++q, i += kBlock) {
      const double zi = z[i];
      const int I = cell_index(zi);
      const double d = (zi - double(I)) - 0.5;
      v[0] += 0.0 * zi;  // NaN for a non-finite position
      if (int(i) + 1 < start[I + 1]) {
        // the particles after this one
        const int lo = start[I];
        Mom4 m = mu[I] - Mom4{1.0, d, d * d, d * d * d};
        if (int(i) > lo) m = m - pre.of(int(i), lo, double(I) + 0.5);
        v[0] += m.m0;
        v[1] += shift1(m, d);
        v[2] += shift2(m, d);
        v[3] += shift3(m, d);
      }
    }
  } else {
    const TriKnots k = tri_knots(W.h[slot], W.L, C);
    const int half = C / 2;
    if (!k.direct) {
      const int last = k.half ? half - 1 : half;
      double a1 = 0.0, a3 = 0.0, b3 = 0.0;
      for (int64_t i = first, q = 0; q < P && i < n; ++q, i += kBlock) {
        const double zi = z[i];
        const int I = cell_index(zi);
        const double ui = zi - double(I);
        KnotPlace g = knot_place(ui, I, k.p1, C, start), h = knot_place(ui, I, k.p2, C, start);
        const Mom4 go = mu[g.J], gp = mu[(I + g.f) & (C - 1)];
        const Mom4 ho = mu[h.J], hp = mu[(I + h.f + (k.image ? 1 : 0)) & (C - 1)];
        while (g.a < g.b || h.a < h.b) {  // both searches at once: their loads overlap
          const int gm = (g.a + g.b) >> 1, hm = (h.a + h.b) >> 1;
          const double gz = g.a < g.b ? z[gm] : 0.0, hz = h.a < h.b ? z[hm] : 0.0;
          if (g.a < g.b) {
            if (gz - g.base < g.t) g.a = gm + 1;
            else g.b = gm;
          }
          if (h.a < h.b) {
            if (hz - h.base < h.t) h.a = hm + 1;
            else h.b = hm;
          }
        }
        double s1, s3, t1, t3;
        before_knot(g, last, go, gp, pre, s1, s3);
        if (k.image)
          t3 = beyond_knot(h, k.p2 > double(h.f), last, ho, hp, pre);
        else
          before_knot(h, last, ho, hp, pre, t1, t3);
        a1 += s1 + 0.0 * zi;
        a3 += s3;
        b3 += t3;
      }
      v[0] = k.s * k.s * k.s * fma(0.125, b3, -0.5 * a3) + 0.0 * a1;
      v[1] = k.s * a1;
    }
    if (k.direct || k.half) {
      const double hs = -0.5 * k.s, period = double(C);
      auto term = [&](double r) {
        const double c = fmax(0.0, fma(-r, k.s, 1.0));
        const double a = fmax(0.0, fma(r, hs, 1.0));
        double kb = fma(-0.5, c * c * c, a * a * a);
        if (k.image) {
          const double ai = fmax(0.0, fma(period - r, hs, 1.0));
          kb = fma(ai * ai, ai, kb);
        }
        v[0] += kb;
        v[1] += c;
      };
      for (int64_t i = first, q = 0; q < P && i < n; ++q, i += kBlock) {
        const double zi = z[i];
        if (k.direct) {
          // the ones behind it, then those of the next period's start: four at a
          // time with the next four in flight (a term beyond the support is 0)
          auto walk = [&](int from, int to, double off) {
            double cur[4], nxt[4];
            auto load = [&](int j, double (&v)[4]) {
#pragma unroll
              for (int u = 0; u < 4; ++u) v[u] = z[min(j + u, to - 1)];
            };
            if (from >= to) return;
            load(from, cur);
            for (int j = from;; j += 4) {
              load(min(j + 4, to - 1), nxt);
#pragma unroll
              for (int u = 0; u < 4; ++u) term(j + u < to ? cur[u] + off : period);
              if (j + 4 >= to || !(cur[3] + off < k.p2)) break;
#pragma unroll
              for (int u = 0; u < 4; ++u) cur[u] = nxt[u];
            }
          };
          walk(int(i) + 1, int(n), -zi);
          if (zi + k.p2 > period) walk(0, int(i), period - zi);
        } else if (cell_index(zi) < half) {  // at half the period each pair once
          const int J = cell_index(zi) + half;
          const double off = double(half) - (zi - double(J - half)) - double(J);
          for (int j = start[J]; j < start[J + 1]; ++j) {
            const double D = z[j] + off;
            term(fmin(D, period - D));
          }
        }
        v[0] += 0.0 * zi;
        v[1] += 0.0 * zi;
      }
    }
  }
  sums_of_block<4, kBlock / 64>(v, red);
  if (threadIdx.x == 0) {
    const bool within = slot == W.B;
    double* o = part + int64_t(slot) * gridDim.x * 2 + int64_t(blockIdx.x) * (within ? 4 : 2);
    o[0] = v[0];
    o[1] = v[1];
    if (within) {
      o[2] = v[2];
      o[3] = v[3];
    }
  }
}

// Band sums Q_m(e), e = 1 + kBands x + wave: the cells' moments in LDS, a lane
// per cell I of the band's pairs (I, I + e mod C), both orders of a pair's
// cells being one band each (e and C - e), so a band up to C / 2 holds every
// unordered pair at e once (at C / 2 twice).
__global__ void __launch_bounds__(kBandBlock) tri_bands_kernel(const Mom4* __restrict__ mu, int C, int emax,
                                                              double* __restrict__ Q) {
  extern __shared__ __align__(16) unsigned char dyn[];
  Mom4* m = reinterpret_cast<Mom4*>(dyn);
#pragma unroll 4
  for (int k = threadIdx.x; k < C; k += kBandBlock) m[k] = mu[k];
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int e = 1 + blockIdx.x * kBands + (threadIdx.x >> 6);
  if (e > emax) return;
  double q0 = 0.0, q1 = 0.0, q2 = 0.0, q3 = 0.0;
#pragma unroll 4
  for (int I = lane; I < C; I += 64) {
    const Mom4 a = m[I], b = m[(I + e) & (C - 1)];
    q0 = fma(a.m0, b.m0, q0);
    q1 += fma(a.m0, b.m1, -(a.m1 * b.m0));
    q2 += fma(a.m0, b.m2, fma(a.m2, b.m0, -2.0 * (a.m1 * b.m1)));
    q3 += fma(a.m0, b.m3, fma(-3.0 * a.m1, b.m2, fma(3.0 * a.m2, b.m1, -(a.m3 * b.m0))));
  }
  q0 = wave_sum(q0);
  q1 = wave_sum(q1);
  q2 = wave_sum(q2);
  q3 = wave_sum(q3);
  if (lane == 0) {
    double* o = Q + 4 * int64_t(e);
    o[0] = q0;
    o[1] = q1;
    o[2] = q2;
    o[3] = q3;
  }
}

// Sums over a band of (4 - 6 u^2 + 3 u^3) / 8 and of (2 - u)^3 / 8, u = u0 + t
// (v - u).
__device__ __forceinline__ double band_inner(double u0, double t, const double (&q)[4]) {
  const double c0 = fma(u0 * u0, fma(3.0, u0, -6.0), 4.0), c1 = u0 * fma(9.0, u0, -12.0), c2 = fma(9.0, u0, -6.0);
  return 0.125 * fma(c0, q[0], t * fma(c1, q[1], t * fma(c2, q[2], 3.0 * t * q[3])));
}
__device__ __forceinline__ double band_outer(double u0, double t, const double (&q)[4]) {
  const double a = 2.0 - u0, a2 = a * a;
  return 0.125 * fma(a2 * a, q[0], t * fma(-3.0 * a2, q[1], t * fma(3.0 * a, q[2], -t * q[3])));
}

// Workgroup b: width b's sums and objective; the last to finish writes the
// first minimum.
__global__ void __launch_bounds__(kBlock) tri_objective_kernel(const double* __restrict__ part, int64_t blocks,
                                                              const double* __restrict__ Q, TriWidths W, double n,
                                                              double* cv, double* __restrict__ sums,
                                                              int32_t* __restrict__ argmin, unsigned int* done) {
  __shared__ double red[kBlock / 64][4];
  __shared__ double vals[KDE_MAX_KAPPAS];
  __shared__ int last;
  const int b = blockIdx.x, B = W.B, C = W.C;
  const TriKnots k = tri_knots(W.h[b], W.L, C);
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  for (int e = 1 + threadIdx.x; e <= W.emax && !k.direct; e += kBlock) {
    if (k.half && 2 * e == C) continue;
    const double w = 2 * e == C ? 0.5 : 1.0, left = double(e - 1);
    const double q[4] = {w * Q[4 * e], w * Q[4 * e + 1], w * Q[4 * e + 2], w * Q[4 * e + 3]};
    const double u0 = double(e) * k.s;
    if (left + 2.0 <= k.p1) {
      v[0] += fmax(0.0, band_inner(u0, k.s, q));
      v[1] += fmax(0.0, fma(1.0 - u0, q[0], -k.s * q[1]));
    } else if (k.image || left + 2.0 <= k.p2) {
      v[0] += fmax(0.0, band_outer(u0, k.s, q));  // (less the power where it holds p1)
    }
    if (k.image && left >= k.p2) v[0] += fmax(0.0, band_outer(double(C - e) * k.s, -k.s, q));
  }
  for (int64_t r = threadIdx.x; r < blocks; r += kBlock) {
    const double* p = part + (int64_t(b) * blocks + r) * 2;
    v[0] += p[0];
    v[1] += p[1];
  }
  if (!k.direct) {  // pairs within a cell: u = |v - u| s <= 1 (their image is a knot's term)
    const double s = k.s, s2 = s * s;
    for (int64_t r = threadIdx.x; r < blocks; r += kBlock) {
      const double* p = part + int64_t(B) * blocks * 2 + r * 4;
      v[0] += 0.125 * fma(3.0 * s2 * s, p[3], fma(-6.0 * s2, p[2], 4.0 * p[0]));
      v[1] += fma(-s, p[1], p[0]);
    }
  }
  sums_of_block<4, kBlock / 64>(v, red);
  if (threadIdx.x == 0) {
    const double h = W.h[b];
    const double S1 = v[0] / (0.75 * h);
    const double S2 = v[1] / h;
    const double val = (n * (2.0 / (3.0 * h)) + 2.0 * S1) / (n * n) - 4.0 * S2 / (n * (n - 1.0));
    __hip_atomic_store(&cv[b], val, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (sums) {
      sums[b] = S1;
      sums[B + b] = S2;
    }
    if (argmin) {
      __threadfence();
      last = atomicAdd(done, 1u) == unsigned(B - 1) ? 1 : 0;
    }
  }
  if (!argmin) return;
  __syncthreads();
  if (!last) return;
  __threadfence();
  if (threadIdx.x < B)
    vals[threadIdx.x] = __hip_atomic_load(&cv[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (threadIdx.x == 0) *argmin = first_min(vals, B);
}

// The arrays of a scan in one block of doubles. They fit the pair layout of the
// same (n, B), whose size the call asks for: the sorted values, and a place of 12
// bytes per particle that holds the unsorted ones with their ranks first, the
// prefix moments then and the band sums last; the counts lie where the cells'
// moments follow.
struct TriBufs {
  Mom4* mu;         // C
  double* sorted;   // n
  double* cells;    // n
  int* rank;        // n
  Mom3* pre;        // ceil(n / 2): over cells and rank
  double* Q;        // 4 (C / 2 + 1): over pre
  int* count;       // C: over mu
  double* part;     // B x blocks x 2, then blocks x 4
  int* start;       // C + 1
  unsigned int* done;
};

int64_t tri_blocks(int64_t n) { return ceil_div(n, (n >= kTriMany ? kTriPer : 1) * kBlock); }

TriBufs carve_tri(Carver& c, int64_t n, int B) {
  const size_t C = size_t(tri_cells(n)), N = size_t(n);
  const size_t part = size_t(tri_blocks(n)) * (2 * size_t(B) + 4), ints = (C + 2 + 1) / 2;
  const size_t shared = std::max(3 * ((N + 1) / 2), 4 * (C / 2 + 1));
  double* base = c.take<double>(4 * C + N + shared + part + ints);
  TriBufs b{};
  if (!base) return b;  // only the size is asked for
  b.mu = reinterpret_cast<Mom4*>(base);
  b.count = reinterpret_cast<int*>(base);
  b.sorted = base + 4 * C;
  b.cells = b.sorted + N;
  b.rank = reinterpret_cast<int*>(b.cells + N);
  b.pre = reinterpret_cast<Mom3*>(b.cells);
  b.Q = b.cells;
  b.part = b.cells + shared;
  b.start = reinterpret_cast<int*>(b.part + part);
  b.done = reinterpret_cast<unsigned int*>(b.start + C + 1);
  return b;
}

}  // namespace

size_t tri_scan_workspace_bytes(int64_t n, int B) {
  Carver c(nullptr, 0);
  carve_tri(c, n, B);
  return c.used;
}

kde_status tri_scan_f64(const kde_domain* dom, int64_t n, const double* x, int B, const double* widths, double* cv,
                        double* sums, int32_t* argmin, void* ws, size_t ws_bytes, hipStream_t s, uint32_t* status) {
  Carver c(ws, ws_bytes);
  const TriBufs b = carve_tri(c, n, B);
  if (!c.fits()) return fail(KDE_E_WORKSPACE, "workspace too small: %zu < %zu bytes", ws_bytes, c.used);
  const int C = tri_cells(n);
  TriWidths W{};
  W.B = B;
  W.C = C;
  W.L = dom->L;
  for (int k = 0; k < B; ++k) W.h[k] = widths[k];
  const double reach = 2.0 * widths[B - 1] / dom->L * double(C) + 2.0;  // bands beyond it are zero for every width
  W.emax = reach < double(C / 2) ? int(reach) : C / 2;
  const int64_t blocks = tri_blocks(n);
  const dim3 per_particle{unsigned(ceil_div(n, kBlock))}, block{unsigned(kBlock)};
  TimedLaunch timed(KDE_KERNEL_CV_PAIRS, s);
  hipExtLaunchKernelGGL(tri_zero_kernel, dim3(unsigned(ceil_div(C, kBlock))), block, 0, s, timed.start(), nullptr, 0,
                        b.count, C, b.done);
  KDE_CHECK_LAUNCH();
  hipLaunchKernelGGL(tri_count_kernel, per_particle, block, 0, s, x, n, dom->L, C, b.count, b.rank, status);
  KDE_CHECK_LAUNCH();
  hipLaunchKernelGGL(tri_scatter_kernel, per_particle, block, 0, s, x, n, dom->L, C, (const int*)b.count,
                     (const int*)b.rank, b.start, b.cells);
  KDE_CHECK_LAUNCH();
  hipLaunchKernelGGL(tri_rank_kernel, per_particle, block, 0, s, (const double*)b.cells, n, (const int*)b.start,
                     b.sorted);
  KDE_CHECK_LAUNCH();
  hipLaunchKernelGGL(tri_prefix_kernel, dim3(unsigned(ceil_div(C, kBlock / 64))), block, 0, s, (const double*)b.sorted,
                     (const int*)b.start, C, b.pre, b.mu);
  KDE_CHECK_LAUNCH();
  const auto knots = n >= kTriMany ? tri_knots_kernel<kTriPer> : tri_knots_kernel<1>;
  hipLaunchKernelGGL(knots, dim3(unsigned(blocks), unsigned(B + 1)), block, 0, s, (const double*)b.sorted, n,
                     (const int*)b.start, (const Mom3*)b.pre, (const Mom4*)b.mu, W, b.part);
  KDE_CHECK_LAUNCH();
  hipLaunchKernelGGL(tri_bands_kernel, dim3(unsigned(ceil_div(W.emax, kBands))), dim3(kBandBlock),
                     size_t(C) * sizeof(Mom4), s, (const Mom4*)b.mu, C, W.emax, b.Q);
  KDE_CHECK_LAUNCH();
  hipExtLaunchKernelGGL(tri_objective_kernel, dim3(unsigned(B)), block, 0, s, nullptr, timed.stop(), 0,
                        (const double*)b.part, blocks, (const double*)b.Q, W, double(n), cv, sums, argmin, b.done);
  KDE_CHECK_LAUNCH();
  return KDE_OK;
}

}  // namespace kde
