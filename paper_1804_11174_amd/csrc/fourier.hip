// Fourier-moment route of the von Mises CV objective (Sec. II.B, Eq.
// cv_def), its Newton refinement in concentration, and the exact pilot at
// the particles for the adaptive widths (Sec. II.C); see kde.h.
//
// On the circle the kernel's Fourier coefficients are rho_m = I_m/I_0, and
// a double sum over pairs of any function of the separation collapses onto
// the sample's moments S_m = sum_j exp(i m theta_j):
//   sum_{i,j} cos(m (theta_i - theta_j)) = |S_m|^2 = P_m.
// So the two sums of the objective cost O(N M) for the moments plus O(M)
// per concentration, instead of O(N^2) per concentration.
//
// Kernels:
//   moments_kernel   -- workgroup (particle chunk, mode block): the chunk's
//                       moments as a matrix product of phases on the FP64
//                       matrix cores (dev_fourier.hpp), into the chunk's
//                       partial rows, which moments_reduce_kernel sums in a
//                       fixed order.
//   series_kernel    -- one workgroup per concentration: the backward
//                       recurrence of the ratios r_m = I_m/I_{m-1},
//                       r_m = kappa / (2 m + kappa r_{m+1}) (stable downwards,
//                       started where the neglected tail has decayed below
//                       e^-40), as a scan of Mobius maps over the workgroup
//                       (series_sums), the ratios multiplied up to rho_m by
//                       a prefix scan, the sums of the series in a fixed
//                       order; the last workgroup takes the first minimum.
//   refine_moments_kernel, refine_series_kernel -- the same for the
//                       refinement, by rotations and in an order of its own.
//   newton_kernel    -- one workgroup: the objective and its derivatives at
//                       the two ends of the bracket around the scan's first
//                       minimum and at the first iterate (the vertex of the
//                       parabola through the three grid values there); from
//                       those, Newton's method on u = log(kappa) with
//                       bisection as the safeguard.
//                       The derivatives come from the same
//                       recurrence differentiated in kappa:
//                         r'_k  = r_k^2 (2k / kappa^2 - r'_{k+1}),
//                         r''_k = 2 r'_k^2 / r_k - r_k^2 (4k / kappa^3 + r''_{k+1}),
//                         rho'_m = rho_m D_m, D_m = sum_{k<=m} r'_k / r_k,
//                         rho''_m = rho_m (D_m^2 + sum_{k<=m} (r''_k / r_k - (r'_k / r_k)^2)).
//                       Each r'_k is positive (I_k/I_{k-1} grows with kappa),
//                       so D_m is a sum of positive terms; the textbook form
//                       rho_{m+1} + (m/kappa) rho_m - rho_1 rho_m is the same
//                       value computed as a difference of O(rho_m) terms,
//                       which loses 2 kappa^2/m^2 rounding units at small m.
//   pilot kernels    -- weights w_m = rho_m(kappa*) S_m (one workgroup), then
//                       the series Re(conj(w_m) e^{i m theta}) at each
//                       particle by Horner's rule in runs of 64 modes, each
//                       run times an exactly reduced phase; logs of the
//                       floored pilot go to a workspace array, their sum
//                       through the fixed-order column sums, then the widths.
// Every reduction has a fixed order: results are deterministic.
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <limits>

#include "dev_fourier.hpp"

namespace kde {

namespace {

constexpr int kPilotRun = 64;           // modes of a Horner run
constexpr int kMaxNewton = 100;
constexpr size_t kNewtonLds = 100 * 1024;  // what the Newton kernels' arrays may take of the LDS
constexpr int kStartEvals = 3;          // refine: bracket ends and first iterate

const int kMaxOrder = fourier_order(KDE_MAX_FOURIER_KAPPA);

// The refinement's own moments (refine_moments_kernel).
constexpr int kRotM = 16;               // consecutive m per group
constexpr int kRotGroups = 2;           // groups per workgroup
constexpr int kRotChunks = 64;          // partials' budget: kRotChunks x kMaxOrder (re, im) pairs
constexpr int64_t kRotBlocks = 4096;    // (chunk, group) pairs a launch aims for
constexpr int kRotPerThread = 8;        // fewest particles per thread

// Partials' budget for N particles, in units of kMaxOrder (re, im) pairs.
int64_t rot_budget(int64_t n) {
  return std::max<int64_t>(1, std::min<int64_t>(kRotChunks, n / (int64_t(kBlock) * kRotPerThread)));
}

// Particle chunks of N particles to order M: about kRotBlocks pairs over the
// ceil(M / kRotM) mode groups, at least kRotPerThread particles per thread,
// and chunks x M within the partials' budget. The sums' order depends on it.
int64_t rot_chunks(int64_t n, int M) {
  int64_t c = ceil_div(kRotBlocks, ceil_div(M, kRotM));
  c = std::min<int64_t>(c, n / (int64_t(kBlock) * kRotPerThread));
  c = std::min<int64_t>(c, rot_budget(n) * kMaxOrder / M);
  return std::max<int64_t>(1, c);
}

// The list with the orders at which the product of Amos's bounds on the
// ratios itself falls below kFourierTail: fourier_order's closed form of that
// product rises by up to 0.051 too far, so it is one higher where its root lies just
// above a whole number, and the refinement's last bits hang on the cut.
FKappas refine_list(const double* k, int B) {
  FKappas f = fourier_list(k, B);
  static const double lim = std::log(kFourierTail);
  for (int b = 0; b < B; ++b) {
    const double below = fourier_root(k[b]) - double(f.order[b] - 1);
    if (!(k[b] > 0.0) || f.order[b] < 2 || below > 0.06) continue;
    double lg = 0.0;
    for (int m = 1; m < f.order[b]; ++m) {
      const double nu = double(m) - 0.5;
      lg += std::log(k[b] / (nu + std::sqrt(nu * nu + k[b] * k[b])));
    }
    if (lg < lim) --f.order[b];
  }
  return f;
}

struct FourierBufs {
  ScanBufs scan;     // partial rows and moments [2 M] (re, im)
  double* rows;      // refine: [chunks][2 M] partial moments, their column sums' scratch
  double* colsum;
  double* S;         // refine: [2 M] moments
  double* rho;       // refine: [3][M + 1], where LDS does not hold them
  double* cvgrid;    // [B]
  double* w;         // [2 M] pilot weights
  double* lf;        // [N] log pilot
  double* bpart;     // [blocks][2]
  double* colsum2;
  double* sums2;     // [2]
};

// Doubles that the column sums of budget x 2 kMaxOrder partials need.
size_t rot_colsum(int64_t budget) {
  return (column_sum_scratch(budget * kMaxOrder, 2) + column_sum_scratch(1, 2 * kMaxOrder)) / sizeof(double) + 1;
}

// What the moments of a scan (or, with B = 1, of the exact pilot) may take, of any
// order: a workspace that does not grow with the order asked for, and holds the
// partials' budget, the sums and a series per concentration of the longest one.
size_t moment_room(int64_t n, int B) {
  Carver c(nullptr, 0);
  const int64_t budget = rot_budget(n);
  c.take<double>(size_t(budget) * 2 * kMaxOrder);
  c.take<double>(rot_colsum(budget));
  c.take<double>(size_t(2) * kMaxOrder);
  c.take<double>(size_t(B) * (kMaxOrder + 1));
  return c.used;
}

// order: that of the moments (their plan depends on it, the size does not).
FourierBufs carve_fourier(Carver& c, int op, int64_t n, int B, int order) {
  FourierBufs b{};
  const int M = kMaxOrder;
  if (op != KDE_OP_CV_REFINE) {
    const size_t room = moment_room(n, op == KDE_OP_ADAPT_EXACT ? 1 : B);
    Carver part(c.take<char>(room), room);
    b.scan = carve_scan(part, room, n, order);
  }
  if (op == KDE_OP_CV_REFINE) {
    // any order's chunks x 2 M partials fit the budget; its column-sum
    // scratch, ceil(chunks / R) x 2 M for R rows per level-1 block, is at
    // most (chunks x 2 M) / R + 2 M
    const int64_t budget = rot_budget(n);
    b.rows = c.take<double>(size_t(budget) * 2 * M);
    b.colsum = c.take<double>(rot_colsum(budget));
    b.S = c.take<double>(size_t(2) * M);
    b.rho = c.take<double>(size_t(3) * (M + 1));
    b.cvgrid = c.take<double>(size_t(B));
  }
  if (op == KDE_OP_ADAPT_EXACT) {
    const int64_t blocks = ceil_div(n, kBlock);
    b.w = c.take<double>(size_t(2) * M);
    b.lf = c.take<double>(size_t(n));
    b.bpart = c.take<double>(size_t(blocks) * 2);
    b.colsum2 = c.take<double>(column_sum_scratch(blocks, 2) / sizeof(double) + 1);
    b.sums2 = c.take<double>(2);
  }
  return b;
}

__device__ __forceinline__ double block_sum(double v, double* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  v = wave_sum(v);
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < kBlock / 64; ++w) t += red[w];
  return t;
}

// Six workgroup sums at once, each in block_sum's order (wave sums, then
// the waves in order), with one exchange through LDS.
__device__ __forceinline__ void block_sum6(double (&v)[6], double (*red)[6]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 6; ++k) v[k] = wave_sum(v[k]);
  __syncthreads();
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < 6; ++k) red[wave][k] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) t += red[w][k];
    v[k] = t;
  }
}

template <typename T>
__global__ void __launch_bounds__(kMomBlock) moments_kernel(const T* __restrict__ x, int64_t n, double L, MomentPlan p,
                                                        double* __restrict__ partials, unsigned int* done,
                                                        uint32_t* status) {
  __shared__ MomSmem sm;
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *done = 0u;
  unit_table_fill(sm.unit);
  __syncthreads();
  moments_unit<T>(x, n, L, p, blockIdx.x, blockIdx.y, partials, sm, status);
}

__global__ void __launch_bounds__(kBlock) moments_reduce_kernel(const double* __restrict__ partials, int64_t rows,
                                                               int cols, double* __restrict__ S) {
  __shared__ double red[kBlock];
  moments_reduce(partials, rows, cols, blockIdx.x, S, red);
}

// The refinement's moments. It reports the number of Newton steps, and the
// last of them are taken at the noise of the objective, so the count hangs on
// every last bit of what it evaluates: with the matrix product's moments,
// which are as exact, it came out one higher or lower for a fifth of random
// samples. The refinement therefore keeps the order of its sums: a thread
// accumulates its particles over kRotM modes by rotation, the threads'
// sums meet in wave_sum's tree and the waves' in order, the chunks' in the
// column sums. What is left to save is around them: the position's phase is
// made once for two groups of modes, and the tree runs over all values at
// once, each exchange halving what a lane holds (63 exchanges for the 64
// values of two groups instead of 384). 65,536 particles to order 911: 33 us
// (47.6 with a group per workgroup and a tree per value).
template <typename T>
__global__ void __launch_bounds__(kBlock) refine_moments_kernel(const T* __restrict__ x, int64_t n, double L, int M,
                                                               int64_t per_chunk, double* __restrict__ rows,
                                                               uint32_t* status) {
  constexpr int kVals = 2 * kRotM;
  __shared__ double red[kRotGroups][kBlock / 64][kVals];
  const int64_t ch = blockIdx.x;
  const int m0 = 1 + int(blockIdx.y) * (kRotM * kRotGroups);
  double v[kRotGroups][kVals];
#pragma unroll
  for (int g = 0; g < kRotGroups; ++g)
#pragma unroll
    for (int k = 0; k < kVals; ++k) v[g][k] = 0.0;
  const int64_t lo = ch * per_chunk, hi = min(n, lo + per_chunk);
  uint32_t* const st = blockIdx.y == 0 ? status : nullptr;  // one column of blocks notes the positions
  for (int64_t j = lo + threadIdx.x; j < hi; j += kBlock) {
    note_numeric(st, !isfinite(double(x[j])), false);
    const double f = wrap_d(double(x[j]), L) / L;
    double c1, s1;
    sincospi(2.0 * f, &s1, &c1);
#pragma unroll
    for (int g = 0; g < kRotGroups; ++g) {
      double c, s;
      phase(m0 + g * kRotM, f, c, s);
#pragma unroll
      for (int k = 0; k < kRotM; ++k) {
        v[g][2 * k] += c;
        v[g][2 * k + 1] += s;
        const double nc = c * c1 - s * s1;
        s = fma(s, c1, c * s1);
        c = nc;
      }
    }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int g = 0; g < kRotGroups; ++g) {
    // after the exchange at distance d a lane keeps the half of the values
    // that its bit d names
    int half = kVals / 2;
#pragma unroll
    for (int d = 32; d >= 2; d >>= 1) {
      const bool up = (lane & d) != 0;
#pragma unroll
      for (int k = 0; k < half; ++k) {
        const double keep = up ? v[g][k + half] : v[g][k];
        const double give = up ? v[g][k] : v[g][k + half];
        v[g][k] = keep + shfl_xor_d(give, d);
      }
      half >>= 1;
    }
    v[g][0] += shfl_xor_d(v[g][0], 1);
    if ((lane & 1) == 0) red[g][wave][lane >> 1] = v[g][0];
  }
  __syncthreads();
  for (int t = threadIdx.x; t < kRotGroups * kVals; t += kBlock) {
    const int g = t / kVals, k = t % kVals;
    const int m = m0 + g * kRotM + (k >> 1);
    if (m <= M) {
      double sum = 0.0;
      for (int w = 0; w < kBlock / 64; ++w) sum += red[g][w][k];
      rows[ch * 2 * int64_t(M) + 2 * (m - 1) + (k & 1)] = sum;
    }
  }
}

// Shared memory of the workgroup-wide series (double-buffered scans).
struct BesselSmem {
  double mat[2][kBlock][4];  // Mobius matrices (row-major 2x2)
  double aff[2][kBlock][2];  // affine maps x -> a + b x
  double pre[2][kBlock][3];  // segment totals (product, sum, sum)
  double red[kBlock / 64];
  double red6[kBlock / 64][6];
};

__device__ __forceinline__ void mat_mul_norm(const double* a, const double* b, double* c) {
  double c0 = fma(a[0], b[0], a[1] * b[2]);
  double c1 = fma(a[0], b[1], a[1] * b[3]);
  double c2 = fma(a[2], b[0], a[3] * b[2]);
  double c3 = fma(a[2], b[1], a[3] * b[3]);
  const double mx = fmax(fmax(fabs(c0), fabs(c1)), fmax(fabs(c2), fabs(c3)));
  const int e = (mx > 0.0) ? ilogb(mx) : 0;  // exact rescaling by a power of two
  c[0] = ldexp(c0, -e);
  c[1] = ldexp(c1, -e);
  c[2] = ldexp(c2, -e);
  c[3] = ldexp(c3, -e);
}

// rho_m(kappa) for m = 0..M into rho[]; with DER also rho'_m, rho''_m into
// d1[], d2[] (kappa > 0 then). All threads of the workgroup take part.
//
// The backward recurrence r_m = kappa / (2m + kappa r_{m+1}), r_{Ms+1} = 0,
// applies the Mobius maps with matrices [[0, kappa], [kappa, 2m]] to the
// homogeneous vector (0, 1): thread t composes the maps of its segment of m
// (non-negative matrices, rescaled by powers of two, so no cancellation), a
// suffix scan over the threads gives every segment the vector entering it
// from above, and each thread walks its segment. r'_m and r''_m obey affine
// recurrences in r'_{m+1} and r''_{m+1} (coefficients from r_m, r'_m), done
// the same way with affine maps; rho_m, D_m and E_m are prefix products and
// sums over m (a combined prefix scan). The composition is a reassociation
// of the recurrence; its rounding grows with the tree depth instead of the
// length of the chain.
// `ratio` (LDS, series_slots doubles) keeps each thread's ratios for its
// later walks (DER only); a scan ends at the last thread that has a run. The
// two forms round the ratio's denominator once (DER) or twice; they always
// have, and the refinement's last bits are kept (refine_moments_kernel).
template <bool DER>
__device__ __forceinline__ void bessel_series(double kappa, int M, double* __restrict__ rho, double* __restrict__ d1,
                                              double* __restrict__ d2, double* __restrict__ ratio, BesselSmem& sm) {
  const int t = threadIdx.x;
  const int Ms = series_length(M, kappa);
  const int len = (Ms + kBlock - 1) / kBlock;
  const int nt = (Ms + len - 1) / len;
  const int lo = 1 + t * len, hi = min(Ms, (t + 1) * len);  // empty when lo > hi
  const double ik2 = DER ? 1.0 / (kappa * kappa) : 0.0;
  const double ik3 = DER ? ik2 / kappa : 0.0;

  // 1. Mobius composition of the segment, suffix scan, then the walk.
  double P[4] = {1.0, 0.0, 0.0, 1.0};
  for (int m = hi; m >= lo; --m) {
    const double Mm[4] = {0.0, kappa, kappa, 2.0 * double(m)};
    double Q[4];
    mat_mul_norm(Mm, P, Q);
    P[0] = Q[0]; P[1] = Q[1]; P[2] = Q[2]; P[3] = Q[3];
  }
  int cur = 0;
  for (int k = 0; k < 4; ++k) sm.mat[0][t][k] = P[k];
  __syncthreads();
  for (int d = 1; d < nt; d <<= 1) {
    if (t + d < kBlock)
      mat_mul_norm(sm.mat[cur][t], sm.mat[cur][t + d], sm.mat[cur ^ 1][t]);
    else
      for (int k = 0; k < 4; ++k) sm.mat[cur ^ 1][t][k] = sm.mat[cur][t][k];
    __syncthreads();
    cur ^= 1;
  }
  const double r_top = (t + 1 < kBlock) ? sm.mat[cur][t + 1][1] / sm.mat[cur][t + 1][3] : 0.0;
  {
    double r = r_top;
    for (int m = hi; m >= lo; --m) {
      r = kappa / (DER ? fma(kappa, r, 2.0 * double(m)) : fma(2.0, double(m), kappa * r));
      if (m <= M) rho[m] = r;
      if (DER) ratio[m] = r;
    }
  }
  double rp_top = 0.0, rpp_top = 0.0;
  if (DER) {
    // 2. r'_m = 2m r_m^2 / kappa^2 - r_m^2 r'_{m+1}.
    double a = 0.0, b = 1.0;
    {
      double r;
      for (int m = hi; m >= lo; --m) {
        r = ratio[m];
        const double r2 = r * r;
        a = fma(-r2, a, 2.0 * double(m) * r2 * ik2);
        b = -r2 * b;
      }
    }
    __syncthreads();  // the matrix scan's reads are done
    sm.aff[0][t][0] = a;
    sm.aff[0][t][1] = b;
    __syncthreads();
    cur = 0;
    for (int d = 1; d < nt; d <<= 1) {
      if (t + d < kBlock) {
        sm.aff[cur ^ 1][t][0] = fma(sm.aff[cur][t][1], sm.aff[cur][t + d][0], sm.aff[cur][t][0]);
        sm.aff[cur ^ 1][t][1] = sm.aff[cur][t][1] * sm.aff[cur][t + d][1];
      } else {
        sm.aff[cur ^ 1][t][0] = sm.aff[cur][t][0];
        sm.aff[cur ^ 1][t][1] = sm.aff[cur][t][1];
      }
      __syncthreads();
      cur ^= 1;
    }
    rp_top = (t + 1 < kBlock) ? sm.aff[cur][t + 1][0] : 0.0;
    // 3. r''_m = 2 r'_m^2 / r_m - r_m^2 (4m / kappa^3 + r''_{m+1}).
    a = 0.0;
    b = 1.0;
    {
      double r, rp = rp_top;
      for (int m = hi; m >= lo; --m) {
        r = ratio[m];
        const double r2 = r * r;
        rp = r2 * (2.0 * double(m) * ik2 - rp);
        const double A = 2.0 * rp * rp / r - 4.0 * double(m) * r2 * ik3;
        a = fma(-r2, a, A);
        b = -r2 * b;
        if (m <= M) d1[m] = rp;
      }
    }
    __syncthreads();
    sm.aff[0][t][0] = a;
    sm.aff[0][t][1] = b;
    __syncthreads();
    cur = 0;
    for (int d = 1; d < nt; d <<= 1) {
      if (t + d < kBlock) {
        sm.aff[cur ^ 1][t][0] = fma(sm.aff[cur][t][1], sm.aff[cur][t + d][0], sm.aff[cur][t][0]);
        sm.aff[cur ^ 1][t][1] = sm.aff[cur][t][1] * sm.aff[cur][t + d][1];
      } else {
        sm.aff[cur ^ 1][t][0] = sm.aff[cur][t][0];
        sm.aff[cur ^ 1][t][1] = sm.aff[cur][t][1];
      }
      __syncthreads();
      cur ^= 1;
    }
    rpp_top = (t + 1 < kBlock) ? sm.aff[cur][t + 1][0] : 0.0;
    {
      double r, rp = rp_top, rpp = rpp_top;
      for (int m = hi; m >= lo; --m) {
        r = ratio[m];
        const double r2 = r * r;
        rp = r2 * (2.0 * double(m) * ik2 - rp);
        rpp = 2.0 * rp * rp / r - r2 * (4.0 * double(m) * ik3 + rpp);
        if (m <= M) d2[m] = rpp;
      }
    }
  }
  // 4. Prefix products and sums over m = 1..M (segments clipped to M).
  const int hm = min(hi, M);
  double sp = 1.0, sD = 0.0, sE = 0.0;
  for (int m = lo; m <= hm; ++m) {
    sp *= rho[m];
    if (DER) {
      const double q = d1[m] / rho[m];
      sD += q;
      sE += d2[m] / rho[m] - q * q;
    }
  }
  __syncthreads();
  sm.pre[0][t][0] = sp;
  sm.pre[0][t][1] = sD;
  sm.pre[0][t][2] = sE;
  __syncthreads();
  cur = 0;
  for (int d = 1; d < nt; d <<= 1) {
    if (t >= d) {
      sm.pre[cur ^ 1][t][0] = sm.pre[cur][t - d][0] * sm.pre[cur][t][0];
      sm.pre[cur ^ 1][t][1] = sm.pre[cur][t - d][1] + sm.pre[cur][t][1];
      sm.pre[cur ^ 1][t][2] = sm.pre[cur][t - d][2] + sm.pre[cur][t][2];
    } else {
      sm.pre[cur ^ 1][t][0] = sm.pre[cur][t][0];
      sm.pre[cur ^ 1][t][1] = sm.pre[cur][t][1];
      sm.pre[cur ^ 1][t][2] = sm.pre[cur][t][2];
    }
    __syncthreads();
    cur ^= 1;
  }
  double p = (t > 0) ? sm.pre[cur][t - 1][0] : 1.0;
  double D = (t > 0) ? sm.pre[cur][t - 1][1] : 0.0;
  double E = (t > 0) ? sm.pre[cur][t - 1][2] : 0.0;
  if (t == 0) rho[0] = 1.0;
  if (DER && t == 0) {
    d1[0] = 0.0;
    d2[0] = 0.0;
  }
  for (int m = lo; m <= hm; ++m) {
    const double rm = rho[m];
    p *= rm;
    rho[m] = p;
    if (DER) {
      const double q = d1[m] / rm;
      D += q;
      E += d2[m] / rm - q * q;
      d1[m] = p * D;
      d2[m] = p * (D * D + E);
    }
  }
  __syncthreads();
}

// Workgroup b: concentration b; the last to finish writes the first minimum.
__global__ void __launch_bounds__(kBlock) series_kernel(const double* __restrict__ S, int M, double n, double L,
                                                       FKappas kap, int Ball, double* cv, double* __restrict__ sums,
                                                       int32_t* __restrict__ argmin, unsigned int* done) {
  __shared__ SeriesSmem sm;
  extern __shared__ __align__(16) double dyn_series[];
  const int b = blockIdx.x;
  const int best = series_unit(kap.k[b], min(M, kap.order[b]), S, n, L, b, gridDim.x, Ball, cv, sums,
                               argmin ? done : nullptr, dyn_series, sm);
  if (best >= 0 && threadIdx.x == 0) *argmin = best;
}

// The refinement's grid of objectives, one workgroup per concentration, with
// its own order of sums too. Dynamic LDS: M + 1 doubles.
__global__ void __launch_bounds__(kBlock) refine_series_kernel(const double* __restrict__ S, int M, double n, double L,
                                                              FKappas kap, double* __restrict__ cv) {
  __shared__ BesselSmem sm;
  extern __shared__ __align__(16) double dyn_series[];
  double* rho = dyn_series;
  const int b = blockIdx.x;
  const int Mb = min(M, kap.order[b]);
  bessel_series<false>(kap.k[b], Mb, rho, nullptr, nullptr, nullptr, sm);
  double a = 0.0, c = 0.0;
  for (int m = 1 + threadIdx.x; m <= Mb; m += kBlock) {
    const double sr = S[2 * (m - 1)], si = S[2 * (m - 1) + 1];
    const double P = fma(sr, sr, si * si);
    const double q = P - n;
    const double r = rho[m];
    a = fma(r * r, P, a);
    c = fma(r, q, c);
  }
  a = block_sum(a, sm.red);
  c = block_sum(c, sm.red);
  if (threadIdx.x == 0) cv[b] = (2.0 * a / (n * n) - 4.0 * c / (n * (n - 1.0)) - 1.0) / L;
}

struct Eval {
  double cv, g, gp;
};

// Objective and its first two derivatives in u = log(kappa), all threads,
// with the series cut at order Mk (that of a kappa at least as large).
__device__ __noinline__ Eval eval_u(double u, const double* __restrict__ S, int Mk, double n, double L, double* rho,
                                       double* d1, double* d2, double* ratio, BesselSmem& sm) {
  const double kappa = exp(u);
  bessel_series<true>(kappa, Mk, rho, d1, d2, ratio, sm);
  double A = 0.0, C = 0.0, A1 = 0.0, C1 = 0.0, A2 = 0.0, C2 = 0.0;
  for (int m = 1 + threadIdx.x; m <= Mk; m += kBlock) {
    const double sr = S[2 * (m - 1)], si = S[2 * (m - 1) + 1];
    const double P = fma(sr, sr, si * si);
    const double q = P - n;
    const double r = rho[m], r1 = d1[m], r2 = d2[m];
    A = fma(r * r, P, A);
    C = fma(r, q, C);
    A1 = fma(2.0 * r * r1, P, A1);
    C1 = fma(r1, q, C1);
    A2 = fma(2.0 * fma(r1, r1, r * r2), P, A2);
    C2 = fma(r2, q, C2);
  }
  double v[6] = {A, C, A1, C1, A2, C2};
  block_sum6(v, sm.red6);
  A = v[0];
  C = v[1];
  A1 = v[2];
  C1 = v[3];
  A2 = v[4];
  C2 = v[5];
  const double n2 = n * n, nn = n * (n - 1.0);
  Eval e;
  e.cv = (2.0 * A / n2 - 4.0 * C / nn - 1.0) / L;
  const double ck = (2.0 * A1 / n2 - 4.0 * C1 / nn) / L;
  const double ckk = (2.0 * A2 / n2 - 4.0 * C2 / nn) / L;
  e.g = kappa * ck;
  e.gp = kappa * kappa * ckk + kappa * ck;
  __syncthreads();  // rho, d1, d2 are rewritten by the next evaluation
  return e;
}

// eval_u by one wave for a series of at most 64 H modes (a run is one mode
// then): lane l holds modes 1 + l + 64 h, and every scan, sum and expression
// is the workgroup form's, on registers and shuffles. No barrier and no LDS
// exchange per scan step: about 7 us against 10.
template <int H>
struct Lanes {
  // o[t] = v[t + d], `rest` past the end
  static __device__ __forceinline__ void down(const double (&v)[H], int d, int lane, double rest, double (&o)[H]) {
    if (d >= 64) {
#pragma unroll
      for (int h = 0; h < H; ++h) {
        o[h] = rest;
#pragma unroll
        for (int k = h + 1; k < H; ++k)
          if (d == 64 * (k - h)) o[h] = v[k];
      }
      return;
    }
    double s[H];
#pragma unroll
    for (int h = 0; h < H; ++h) s[h] = __shfl(v[h], (lane + d) & 63, 64);
#pragma unroll
    for (int h = 0; h < H; ++h) o[h] = lane + d < 64 ? s[h] : (h + 1 < H ? s[(h + 1) % H] : rest);
  }
  // o[t] = v[t - d], `rest` before the start
  static __device__ __forceinline__ void up(const double (&v)[H], int d, int lane, double rest, double (&o)[H]) {
    if (d >= 64) {
#pragma unroll
      for (int h = 0; h < H; ++h) {
        o[h] = rest;
#pragma unroll
        for (int k = 0; k < h; ++k)
          if (d == 64 * (h - k)) o[h] = v[k];
      }
      return;
    }
    double s[H];
#pragma unroll
    for (int h = 0; h < H; ++h) s[h] = __shfl(v[h], (lane - d) & 63, 64);
#pragma unroll
    for (int h = 0; h < H; ++h) o[h] = lane >= d ? s[h] : (h > 0 ? s[(h + H - 1) % H] : rest);
  }
};

// Suffix scan of the affine maps x -> a + b x; a[t + 1] into top.
template <int H>
__device__ __forceinline__ void affine_tops(double (&a)[H], double (&b)[H], int nt, int lane, double (&top)[H]) {
  for (int d = 1; d < nt; d <<= 1) {
    double oa[H], ob[H];
    Lanes<H>::down(a, d, lane, 0.0, oa);
    Lanes<H>::down(b, d, lane, 1.0, ob);
#pragma unroll
    for (int h = 0; h < H; ++h) {
      a[h] = fma(b[h], oa[h], a[h]);
      b[h] = b[h] * ob[h];
    }
  }
  Lanes<H>::down(a, 1, lane, 0.0, top);
}

template <int H>
__device__ __noinline__ Eval eval_wave(double u, const double* __restrict__ power, int Mk, double n, double L) {
  const double kappa = exp(u);
  const int lane = threadIdx.x & 63;
  const int nt = series_length(Mk, kappa);
  const double ik2 = 1.0 / (kappa * kappa);
  const double ik3 = ik2 / kappa;
  double pa[H], pb[H], pc[H], pd[H];
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int m = 1 + lane + 64 * h;
    const Mat2 P = m <= nt ? mat_norm(Mat2{0.0, kappa, kappa, 2.0 * double(m)}) : Mat2{1.0, 0.0, 0.0, 1.0};
    pa[h] = P.a;
    pb[h] = P.b;
    pc[h] = P.c;
    pd[h] = P.d;
  }
  for (int d = 1; d < nt; d <<= 1) {
    double qa[H], qb[H], qc[H], qd[H];
    Lanes<H>::down(pa, d, lane, 1.0, qa);
    Lanes<H>::down(pb, d, lane, 0.0, qb);
    Lanes<H>::down(pc, d, lane, 0.0, qc);
    Lanes<H>::down(pd, d, lane, 1.0, qd);
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const Mat2 P = mat_mul(Mat2{pa[h], pb[h], pc[h], pd[h]}, Mat2{qa[h], qb[h], qc[h], qd[h]});
      pa[h] = P.a;
      pb[h] = P.b;
      pc[h] = P.c;
      pd[h] = P.d;
    }
  }
  double top[H], r[H], a[H], b[H];
#pragma unroll
  for (int h = 0; h < H; ++h) a[h] = pb[h] / pd[h];
  Lanes<H>::down(a, 1, lane, 0.0, top);
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int m = 1 + lane + 64 * h;
    const bool in = m <= nt;
    r[h] = kappa / fma(kappa, top[h], 2.0 * double(m));
    const double r2 = r[h] * r[h];
    a[h] = in ? 2.0 * double(m) * r2 * ik2 : 0.0;
    b[h] = in ? -r2 : 1.0;
  }
  affine_tops<H>(a, b, nt, lane, top);
  double rp[H];
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int m = 1 + lane + 64 * h;
    const bool in = m <= nt;
    const double r2 = r[h] * r[h];
    rp[h] = r2 * (2.0 * double(m) * ik2 - top[h]);
    const double A = 2.0 * rp[h] * rp[h] / r[h] - 4.0 * double(m) * r2 * ik3;
    a[h] = in ? A : 0.0;
    b[h] = in ? -r2 : 1.0;
  }
  affine_tops<H>(a, b, nt, lane, top);
  double q[H], e[H], sp[H], sD[H], sE[H];
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int m = 1 + lane + 64 * h;
    const bool in = m <= Mk;
    const double r2 = r[h] * r[h];
    const double rpp = 2.0 * rp[h] * rp[h] / r[h] - r2 * (4.0 * double(m) * ik3 + top[h]);
    q[h] = rp[h] / r[h];
    e[h] = rpp / r[h] - q[h] * q[h];
    sp[h] = in ? r[h] : 1.0;
    sD[h] = in ? q[h] : 0.0;
    sE[h] = in ? e[h] : 0.0;
  }
  for (int d = 1; d < nt; d <<= 1) {
    double op[H], oD[H], oE[H];
    Lanes<H>::up(sp, d, lane, 1.0, op);
    Lanes<H>::up(sD, d, lane, 0.0, oD);
    Lanes<H>::up(sE, d, lane, 0.0, oE);
#pragma unroll
    for (int h = 0; h < H; ++h) {
      sp[h] = op[h] * sp[h];
      sD[h] = oD[h] + sD[h];
      sE[h] = oE[h] + sE[h];
    }
  }
  double p[H], D[H], E[H];
  Lanes<H>::up(sp, 1, lane, 1.0, p);
  Lanes<H>::up(sD, 1, lane, 0.0, D);
  Lanes<H>::up(sE, 1, lane, 0.0, E);
  double v[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int m = 1 + lane + 64 * h;
    double t[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (m <= Mk) {
      const double rm = p[h] * r[h];
      D[h] += q[h];
      E[h] += e[h];
      const double r1 = rm * D[h], r2 = rm * (D[h] * D[h] + E[h]);
      const double P = power[m], w = P - n;
      t[0] = (rm * rm) * P;
      t[1] = rm * w;
      t[2] = (2.0 * rm * r1) * P;
      t[3] = r1 * w;
      t[4] = (2.0 * fma(r1, r1, rm * r2)) * P;
      t[5] = r2 * w;
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] += wave_sum(t[k]);
  }
  const double n2 = n * n, nn = n * (n - 1.0);
  Eval o;
  o.cv = (2.0 * v[0] / n2 - 4.0 * v[1] / nn - 1.0) / L;
  const double ck = (2.0 * v[2] / n2 - 4.0 * v[3] / nn) / L;
  const double ckk = (2.0 * v[4] / n2 - 4.0 * v[5] / nn) / L;
  o.g = kappa * ck;
  o.gp = kappa * kappa * ckk + kappa * ck;
  return o;
}

// The refinement's bracket: the list neighbours of the scan's first
// minimum bs (the lower one replaced by the first positive kappa when it is
// 0), the series order Mk of its upper end, and the first Newton iterate:
// the vertex of the parabola through the three grid values around bs in
// u = log(kappa) when it lies inside the bracket, else log(kappa_bs), else
// the bracket's middle. valid is false when there is no bracket of
// positive concentrations.
struct Bracket {
  int bs, Mk;
  double klo, khi, ul, uh, u0;
  bool valid;
};

__device__ Bracket make_bracket(const double* __restrict__ cvgrid, int B, const FKappas& kap, int M) {
  Bracket r;
  r.bs = first_min(cvgrid, B);
  r.Mk = min(M, kap.order[min(r.bs + 1, B - 1)]);
  double klo = kap.k[max(r.bs - 1, 0)];
  const double khi = kap.k[min(r.bs + 1, B - 1)];
  if (!(klo > 0.0)) {
    double kp = 0.0;
    for (int t = 0; t < B; ++t)
      if (kap.k[t] > 0.0) {
        kp = kap.k[t];
        break;
      }
    klo = kp;
  }
  r.valid = (klo > 0.0) && (khi > klo);
  r.klo = klo;
  r.khi = khi;
  r.ul = r.valid ? log(klo) : 0.0;
  r.uh = r.valid ? log(khi) : 0.0;
  r.u0 = 0.5 * (r.ul + r.uh);
  const int b = r.bs;
  if (r.valid && b > 0 && b < B - 1 && kap.k[b] > klo && kap.k[b] < khi) {
    const double ub = log(kap.k[b]);
    r.u0 = ub;
    if (kap.k[b - 1] > 0.0) {
      const double ua = log(kap.k[b - 1]), uc = log(kap.k[b + 1]);
      const double p = (ub - ua) * (cvgrid[b] - cvgrid[b + 1]);
      const double q = (ub - uc) * (cvgrid[b] - cvgrid[b - 1]);
      const double den = p - q;
      if (den != 0.0) {
        const double uv = ub - 0.5 * ((ub - ua) * p - (ub - uc) * q) / den;
        if (uv > r.ul && uv < r.uh) r.u0 = uv;
      }
    }
  }
  return r;
}

// result: [kappa*, cv(kappa*), dCV/du at kappa*, steps, b*], by one workgroup.
// A bracket whose series has at most 256 modes (kappa* up to a few hundred): waves
// 0, 1 and 2 evaluate its ends and the first iterate side by side, then wave 0
// goes on alone; a longer one is evaluated by the whole workgroup, one point
// after the other. Dynamic LDS: the ratios of the series (series_slots)
// and, where they fit (LDS), three arrays of M + 1.
// 65,536 particles, 32 concentrations up to 1e4 (911 modes, the bracket's series
// about 90): 49 us, 62 with a workgroup for each start and another for the steps.
template <bool LDS>
__global__ void __launch_bounds__(kBlock) newton_kernel(const double* __restrict__ S, int M, double n, double L,
                                                       FKappas kap, int B, const double* __restrict__ cvgrid,
                                                       double* __restrict__ rho3, double* __restrict__ result,
                                                       int32_t* __restrict__ argmin) {
  __shared__ BesselSmem sm;
  __shared__ double power[kBlock + 1];
  __shared__ Eval start[kStartEvals];
  extern __shared__ __align__(16) double dyn_series[];
  double* rho = LDS ? dyn_series : rho3;
  double* d1 = rho + (M + 1);
  double* d2 = rho + 2 * (M + 1);
  double* ratio = LDS ? dyn_series + 3 * size_t(M + 1) : dyn_series;
  const int wave = threadIdx.x >> 6;
  const Bracket br = make_bracket(cvgrid, B, kap, M);
  const int bs = br.bs;
  if (argmin && threadIdx.x == 0) *argmin = bs;
  double k_best = 0.0, cv_best = 0.0, g_best = 0.0;
  int steps = 0;
  if (!br.valid) {
    // no bracket of positive concentrations: the scan's value
    k_best = kap.k[bs];
    cv_best = cvgrid[bs];
    g_best = 0.0;
  } else {
    const int modes = series_slots(br.Mk, br.khi) - 1;  // the longest series of the bracket
    const bool alone = modes <= kBlock;
    if (alone && int(threadIdx.x) < br.Mk) {
      const double sr = S[2 * threadIdx.x], si = S[2 * threadIdx.x + 1];
      power[threadIdx.x + 1] = fma(sr, sr, si * si);
    }
    __syncthreads();
    auto eval = [&](double u) {
      if (!alone) return eval_u(u, S, br.Mk, n, L, rho, d1, d2, ratio, sm);
      return modes <= 128 ? eval_wave<2>(u, power, br.Mk, n, L) : eval_wave<4>(u, power, br.Mk, n, L);
    };
    // the starts: side by side, or one after the other
    for (int k = alone ? wave : 0; k < kStartEvals; k += alone ? kBlock / 64 : 1) {
      const Eval e = eval(k == 0 ? br.ul : (k == 1 ? br.uh : br.u0));
      if (alone ? (threadIdx.x & 63) == 0 : threadIdx.x == 0) start[k] = e;
    }
    __syncthreads();
    if (alone && wave != 0) return;  // (no barrier follows)
    double ul = br.ul, uh = br.uh;
    const Eval el = start[0], eh = start[1];
    steps = 2;
    if (!(el.g < 0.0 && eh.g > 0.0)) {
      const bool lo_wins = el.cv <= eh.cv;
      k_best = lo_wins ? br.klo : br.khi;
      cv_best = lo_wins ? el.cv : eh.cv;
      g_best = lo_wins ? el.g : eh.g;
    } else {
      double u = br.u0;
      Eval e = start[2];
      ++steps;
      for (int it = 0; it < kMaxNewton && e.g != 0.0; ++it) {
        if (e.g < 0.0)
          ul = u;
        else
          uh = u;
        double un = u - e.g / e.gp;
        if (!(e.gp > 0.0) || !(un > ul && un < uh)) un = 0.5 * (ul + uh);
        const bool done = fabs(un - u) <= 1e-14 * fmax(1.0, fabs(un)) || (uh - ul) <= 1e-14 * fmax(1.0, fabs(un));
        u = un;
        e = eval(u);
        ++steps;
        if (done) break;
      }
      k_best = exp(u);
      cv_best = e.cv;
      g_best = e.g;
    }
  }
  if (threadIdx.x == 0) {
    result[0] = k_best;
    result[1] = cv_best;
    result[2] = g_best;
    result[3] = double(steps);
    result[4] = double(bs);
  }
}

// w_m = rho_m(kappa) S_m, m = 1..M (one workgroup; dynamic LDS: series_lds).
__global__ void __launch_bounds__(kBlock) pilot_weights_kernel(const double* __restrict__ S, int M, double kappa,
                                                              double* __restrict__ w) {
  __shared__ ScanSmem sm;
  extern __shared__ __align__(16) double dyn_series[];
  series_rho(kappa, M, dyn_series, sm);
  for (int m = 1 + threadIdx.x; m <= M; m += kBlock) {
    w[2 * (m - 1)] = dyn_series[m] * S[2 * (m - 1)];
    w[2 * (m - 1) + 1] = dyn_series[m] * S[2 * (m - 1) + 1];
  }
}

// Per particle: f = (1/L)(1 + (2/N) sum_m Re(conj(w_m) e^{i m theta})),
// floored at `floor`; lf[i] = log f; block sums of (log f, floored).
//
// The series by Horner's rule in e^{i theta}, X <- X e^{i theta} + conj(w_m)
// downwards: 4 multiply-adds a mode, in runs of kPilotRun modes that each
// are multiplied by a phase of their own, so the rounding of e^{i theta} is
// raised to no higher power. 1,000,003 floats at 46 modes: 19.3 us (33.5 with 6
// operations a mode, 21 with the library's logarithm, two divisions and one
// particle per thread). A sum over all workgroups by the last one to finish
// instead of the column sums' two launches was 25 us slower: each workgroup's
// fence writes its logarithms back.
template <typename T, int P>
__global__ void __launch_bounds__(kBlock) pilot_kernel(const T* __restrict__ x, int64_t n, double L, int M,
                                                      const double2* __restrict__ w, double floor_v,
                                                      double* __restrict__ lf, double* __restrict__ bpart,
                                                      uint32_t* status) {
  __shared__ double red[kBlock / 64];
  __shared__ double2 unit[256];
  const int64_t base = int64_t(blockIdx.x) * (P * kBlock) + threadIdx.x;
  const double inv_L = 1.0 / L, two_n = 2.0 / double(n);
  T xv[P];
#pragma unroll
  for (int p = 0; p < P; ++p) xv[p] = x[min(base + p * kBlock, n - 1)];
  unit_table_fill(unit);
  __syncthreads();
  double f[P], acc[P];
  double2 z1[P];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    note_numeric(status, !isfinite(double(xv[p])), false);
    f[p] = period_fraction(double(xv[p]), L, inv_L);
    z1[p] = table_phase(1.0, f[p], unit);
    acc[p] = 0.0;
  }
  for (int m0 = 1 + (M - 1) / kPilotRun * kPilotRun; m0 >= 1; m0 -= kPilotRun) {
    double xr[P], xi[P];
#pragma unroll
    for (int p = 0; p < P; ++p) xr[p] = xi[p] = 0.0;
    auto mode = [&](int m) {
      const double2 a = w[m - 1];
#pragma unroll
      for (int p = 0; p < P; ++p) {
        const double r = fma(xr[p], z1[p].x, fma(-xi[p], z1[p].y, a.x));
        xi[p] = fma(xr[p], z1[p].y, fma(xi[p], z1[p].x, -a.y));
        xr[p] = r;
      }
    };
    int m = min(M, m0 + kPilotRun - 1);
    for (; (m - m0 + 1) & 7; --m) mode(m);
    for (; m >= m0; m -= 8) {
#pragma unroll
      for (int u = 0; u < 8; ++u) mode(m - u);
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const double2 z = m0 == 1 ? z1[p] : table_phase(double(m0), f[p], unit);
      acc[p] = fma(xr[p], z.x, fma(-xi[p], z.y, acc[p]));
    }
  }
  double lsum = 0.0, fl = 0.0;
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int64_t i = base + p * kBlock;
    double v = fma(acc[p], two_n, 1.0) * inv_L;
    bool low = false;
    if (!(v >= floor_v)) {  // also catches NaN: floored and counted
      low = true;
      v = isnan(v) ? v : floor_v;
    }
    const double l = log_normal(v);
    if (i < n) {
      lf[i] = l;
      lsum += l;
      fl += low ? 1.0 : 0.0;
    }
  }
  lsum = block_sum(lsum, red);
  fl = block_sum(fl, red);
  if (threadIdx.x == 0) {
    bpart[2 * int64_t(blockIdx.x)] = lsum;
    bpart[2 * int64_t(blockIdx.x) + 1] = fl;
  }
}

template <typename T>
__global__ void __launch_bounds__(kBlock) pilot_apply_kernel(const double* __restrict__ lf, int64_t n,
                                                            double kappa_star, double alpha,
                                                            const double* __restrict__ sums, T* __restrict__ kout,
                                                            double* __restrict__ log_g_out,
                                                            int64_t* __restrict__ nfl_out) {
  const double log_g = sums[0] / double(n);
  const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (i < n) kout[i] = T(kappa_star * exp(2.0 * alpha * (lf[i] - log_g)));
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (log_g_out) *log_g_out = log_g;
    if (nfl_out) *nfl_out = int64_t(sums[1]);
  }
}

kde_status moments_any(const kde_domain* dom, int64_t n, const void* x, const FourierBufs& b, hipStream_t s) {
  TimedLaunch timed(KDE_KERNEL_MOMENTS, s);
  if (dom->prec == KDE_F64)
    return launch_moments(static_cast<const double*>(x), n, dom->L, b.scan, s, timed.start(), timed.stop(),
                          plain_numeric_word());
  return launch_moments(static_cast<const float*>(x), n, dom->L, b.scan, s, timed.start(), timed.stop(),
                        plain_numeric_word());
}

template <typename T>
kde_status refine_moments(const T* x, int64_t n, double L, int M, const FourierBufs& b, hipStream_t s) {
  const int64_t chunks = rot_chunks(n, M);
  const dim3 grid{unsigned(chunks), unsigned(ceil_div(M, kRotM * kRotGroups))};
  {
    TimedLaunch timed(KDE_KERNEL_MOMENTS, s);
    hipExtLaunchKernelGGL(refine_moments_kernel<T>, grid, dim3(kBlock), 0, s, timed.start(), timed.stop(), 0, x, n, L, M,
                          ceil_div(n, chunks), b.rows, plain_numeric_word());
  }
  KDE_CHECK_LAUNCH();
  return launch_column_sum(b.rows, chunks, 2 * M, b.colsum, b.S, s);
}

template <bool LDS>
kde_status launch_newton(size_t lds, const FourierBufs& b, int M, double n, double L, const FKappas& kl, int B,
                         const double* grid, double* result, int32_t* argmin, hipStream_t s) {
  hipLaunchKernelGGL(newton_kernel<LDS>, dim3(1), dim3(kBlock), lds, s, (const double*)b.S, M, n, L, kl, B, grid,
                     b.rho, result, argmin);
  KDE_CHECK_LAUNCH();
  return KDE_OK;
}

// Four particles per thread once two workgroups per CU are left (they share the
// table, the scalars and the sums): 1,000,003 particles 52.9 us with the other
// kernels against 56.6; 20,000 are 4 us slower, bound by the latency of a wave.
constexpr int64_t kPilotWide = 4 * int64_t(kBlock) * 2 * 256;

template <typename T>
kde_status launch_pilot(const T* x, int64_t n, double L, int M, const FourierBufs& b, hipStream_t s, hipEvent_t t0,
                        int64_t& blocks) {
  const double floor_v = double(std::numeric_limits<T>::min());
  const double2* w = reinterpret_cast<const double2*>(b.w);
  blocks = ceil_div(n, (n >= kPilotWide ? 4 : 1) * kBlock);
  const dim3 grid{unsigned(blocks)};
  if (n >= kPilotWide)
    hipExtLaunchKernelGGL((pilot_kernel<T, 4>), grid, dim3(kBlock), 0, s, t0, nullptr, 0, x, n, L, M, w, floor_v, b.lf,
                          b.bpart, plain_numeric_word());
  else
    hipExtLaunchKernelGGL((pilot_kernel<T, 1>), grid, dim3(kBlock), 0, s, t0, nullptr, 0, x, n, L, M, w, floor_v, b.lf,
                          b.bpart, plain_numeric_word());
  KDE_CHECK_LAUNCH();
  return KDE_OK;
}

kde_status check_fourier_common(const kde_domain* dom, int64_t N, const void* x, int64_t nmin) {
  KDE_RETURN_IF(check_domain(dom, false));
  if (dom->shape != KDE_SHAPE_VONMISES) return fail(KDE_E_INVALID_ARG, "the Fourier route is defined for the von Mises shape");
  if (N < nmin || N > kMaxN) return fail(KDE_E_INVALID_ARG, "N must lie in [%lld, %lld] (got %lld)", (long long)nmin, (long long)kMaxN, (long long)N);
  if (!x) return fail(KDE_E_INVALID_ARG, "x must not be NULL");
  return KDE_OK;
}

kde_status check_fourier_kappas(int B, const double* kappas_h) {
  if (B < 1 || B > KDE_MAX_KAPPAS) return fail(KDE_E_INVALID_ARG, "B must lie in [1, %d] (got %d)", KDE_MAX_KAPPAS, B);
  if (!kappas_h) return fail(KDE_E_INVALID_ARG, "kappas_h is NULL");
  for (int b = 0; b < B; ++b) {
    const double k = kappas_h[b];
    if (!std::isfinite(k) || k < 0.0 || k > KDE_MAX_FOURIER_KAPPA)
      return fail(KDE_E_INVALID_ARG, "every kappa must lie in [0, %g] (got %g at %d)", KDE_MAX_FOURIER_KAPPA, k, b);
    if (b > 0 && !(k > kappas_h[b - 1])) return fail(KDE_E_INVALID_ARG, "kappas must be strictly ascending (index %d)", b);
  }
  return KDE_OK;
}

}  // namespace

template <typename T>
kde_status launch_moment_rows(const T* x, int64_t n, double L, const ScanBufs& b, hipStream_t s, hipEvent_t t0,
                              hipEvent_t t1, uint32_t* status) {
  const MomentPlan& p = b.plan;
  hipExtLaunchKernelGGL((moments_kernel<T>), dim3(unsigned(p.chunks), unsigned(p.mblocks)), dim3(kMomBlock), 0, s, t0,
                        t1, 0, x, n, L, p, b.partials, b.done, status);
  KDE_CHECK_LAUNCH();
  return KDE_OK;
}
template kde_status launch_moment_rows<double>(const double*, int64_t, double, const ScanBufs&, hipStream_t,
                                               hipEvent_t, hipEvent_t, uint32_t*);

template <typename T>
kde_status launch_moments(const T* x, int64_t n, double L, const ScanBufs& b, hipStream_t s, hipEvent_t t0,
                          hipEvent_t t1, uint32_t* status) {
  const MomentPlan& p = b.plan;
  const bool one = p.rows == 1;  // (the moments themselves: partials is S)
  KDE_RETURN_IF(launch_moment_rows(x, n, L, b, s, t0, one ? t1 : nullptr, status));
  if (one) return KDE_OK;
  hipExtLaunchKernelGGL(moments_reduce_kernel, dim3(unsigned(ceil_div(2 * p.M, kRedCols))), dim3(kBlock), 0, s, nullptr,
                        t1, 0, (const double*)b.partials, p.rows, 2 * p.M, b.S);
  KDE_CHECK_LAUNCH();
  return KDE_OK;
}
template kde_status launch_moments<double>(const double*, int64_t, double, const ScanBufs&, hipStream_t, hipEvent_t,
                                           hipEvent_t, uint32_t*);
template kde_status launch_moments<float>(const float*, int64_t, double, const ScanBufs&, hipStream_t, hipEvent_t,
                                          hipEvent_t, uint32_t*);

kde_status launch_series(const ScanBufs& b, int M, int64_t n, double L, const FKappas& kap, int B, int Ball,
                         double* cv, double* sums, int32_t* argmin, hipStream_t s, hipEvent_t t1) {
  hipExtLaunchKernelGGL(series_kernel, dim3(unsigned(B)), dim3(kBlock), series_lds(M), s, nullptr, t1, 0,
                        (const double*)b.S, M, double(n), L, kap, Ball, cv, sums, argmin, b.done);
  KDE_CHECK_LAUNCH();
  return KDE_OK;
}

size_t fourier_workspace_bytes(int op, int64_t n, int B) {
  Carver c(nullptr, 0);
  carve_fourier(c, op, n, B, kMaxOrder);
  return c.used;
}

}  // namespace kde

using namespace kde;

extern "C" {

kde_status kde_cv_scan_fourier(const kde_domain* dom, int64_t N, const void* x, int32_t B, const double* kappas_h,
                               double* cv, double* sums, int32_t* argmin, void* ws, size_t ws_bytes, void* stream) {
  clear_error();
  KDE_RETURN_IF(check_fourier_common(dom, N, x, 2));
  KDE_RETURN_IF(check_fourier_kappas(B, kappas_h));
  if (!cv) return fail(KDE_E_INVALID_ARG, "cv must not be NULL");
  KDE_RETURN_IF(check_workspace(ws, ws_bytes, fourier_workspace_bytes(KDE_OP_CV_FOURIER, N, B)));
  hipStream_t s = static_cast<hipStream_t>(stream);
  Carver c(ws, ws_bytes);
  const int M = fourier_order(kappas_h[B - 1]);
  const FourierBufs b = carve_fourier(c, KDE_OP_CV_FOURIER, N, B, M);
  KDE_RETURN_IF(moments_any(dom, N, x, b, s));
  return launch_series(b.scan, M, N, dom->L, fourier_list(kappas_h, B), B, B, cv, sums, argmin, s, nullptr);
}

kde_status kde_cv_refine(const kde_domain* dom, int64_t N, const void* x, int32_t B, const double* kappas_h,
                         double* result, double* cv, int32_t* argmin, void* ws, size_t ws_bytes, void* stream) {
  clear_error();
  KDE_RETURN_IF(check_fourier_common(dom, N, x, 2));
  KDE_RETURN_IF(check_fourier_kappas(B, kappas_h));
  if (!result) return fail(KDE_E_INVALID_ARG, "result must not be NULL");
  KDE_RETURN_IF(check_workspace(ws, ws_bytes, fourier_workspace_bytes(KDE_OP_CV_REFINE, N, B)));
  hipStream_t s = static_cast<hipStream_t>(stream);
  Carver c(ws, ws_bytes);
  const FourierBufs b = carve_fourier(c, KDE_OP_CV_REFINE, N, B, 0);
  const FKappas kl = refine_list(kappas_h, B);
  const int M = kl.order[B - 1];
  if (dom->prec == KDE_F64)
    KDE_RETURN_IF(refine_moments(static_cast<const double*>(x), N, dom->L, M, b, s));
  else
    KDE_RETURN_IF(refine_moments(static_cast<const float*>(x), N, dom->L, M, b, s));
  double* grid = cv ? cv : b.cvgrid;
  hipLaunchKernelGGL(refine_series_kernel, dim3(unsigned(B)), dim3(kBlock), sizeof(double) * size_t(M + 1), s,
                     (const double*)b.S, M, double(N), dom->L, kl, grid);
  KDE_CHECK_LAUNCH();
  const size_t ratios = sizeof(double) * size_t(series_slots(M, kappas_h[B - 1]));
  const size_t all = ratios + sizeof(double) * 3 * size_t(M + 1);
  if (all <= kNewtonLds) {
    KDE_RETURN_IF(check_lds(all + sizeof(BesselSmem)));
    return launch_newton<true>(all, b, M, double(N), dom->L, kl, B, grid, result, argmin, s);
  }
  KDE_RETURN_IF(check_lds(ratios + sizeof(BesselSmem)));
  return launch_newton<false>(ratios, b, M, double(N), dom->L, kl, B, grid, result, argmin, s);
}

kde_status kde_adapt_widths_exact(const kde_domain* dom, int64_t N, const void* x, double kappa_star, double alpha,
                                  void* kappa_out, double* log_geomean, int64_t* n_floored, void* ws, size_t ws_bytes,
                                  void* stream) {
  clear_error();
  KDE_RETURN_IF(check_fourier_common(dom, N, x, 1));
  if (!kappa_out) return fail(KDE_E_INVALID_ARG, "kappa_out must not be NULL");
  if (!std::isfinite(kappa_star) || !(kappa_star > 0.0) || kappa_star > KDE_MAX_FOURIER_KAPPA)
    return fail(KDE_E_INVALID_ARG, "kappa_star must lie in (0, %g] (got %g)", KDE_MAX_FOURIER_KAPPA, kappa_star);
  if (!std::isfinite(alpha) || alpha < 0.0) return fail(KDE_E_INVALID_ARG, "alpha must be finite and >= 0 (got %g)", alpha);
  KDE_RETURN_IF(check_workspace(ws, ws_bytes, fourier_workspace_bytes(KDE_OP_ADAPT_EXACT, N, 0)));
  hipStream_t s = static_cast<hipStream_t>(stream);
  Carver c(ws, ws_bytes);
  const int M = fourier_order(kappa_star);
  const FourierBufs b = carve_fourier(c, KDE_OP_ADAPT_EXACT, N, 0, M);
  KDE_RETURN_IF(moments_any(dom, N, x, b, s));
  hipLaunchKernelGGL(pilot_weights_kernel, dim3(1), dim3(kBlock), series_lds(M), s, (const double*)b.scan.S, M,
                     kappa_star, b.w);
  KDE_CHECK_LAUNCH();
  TimedLaunch timed(KDE_KERNEL_ADAPT, s);  // from the pilot values' start to the widths' end
  int64_t blocks = 0;
  if (dom->prec == KDE_F64)
    KDE_RETURN_IF(launch_pilot(static_cast<const double*>(x), N, dom->L, M, b, s, timed.start(), blocks));
  else
    KDE_RETURN_IF(launch_pilot(static_cast<const float*>(x), N, dom->L, M, b, s, timed.start(), blocks));
  KDE_RETURN_IF(launch_column_sum(b.bpart, blocks, 2, b.colsum2, b.sums2, s));
  const dim3 grid{unsigned(ceil_div(N, kBlock))};
  if (dom->prec == KDE_F64)
    hipExtLaunchKernelGGL(pilot_apply_kernel<double>, grid, dim3(kBlock), 0, s, nullptr, timed.stop(), 0,
                          (const double*)b.lf, N, kappa_star, alpha, (const double*)b.sums2,
                          static_cast<double*>(kappa_out), log_geomean, n_floored);
  else
    hipExtLaunchKernelGGL(pilot_apply_kernel<float>, grid, dim3(kBlock), 0, s, nullptr, timed.stop(), 0,
                          (const double*)b.lf, N, kappa_star, alpha, (const double*)b.sums2,
                          static_cast<float*>(kappa_out), log_geomean, n_floored);
  KDE_CHECK_LAUNCH();
  return KDE_OK;
}

}  // extern "C"
