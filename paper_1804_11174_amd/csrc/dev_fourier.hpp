#pragma once
// Device pieces of the Fourier-moment evaluation of the von Mises CV
// objective (Sec. II.B, Eq. cv_def), shared by the CV scan (cv.hip), the
// Fourier entry points (fourier.hip) and the batched engine (batch.hip):
// the moments of the particle angles and the series over them.
//
// Moments S_m = sum_j exp(i m theta_j), m = 1..M, theta = 2 pi x / L. With a
// step s and m = s a + b or s a - b, 0 <= b <= (s - 1) / 2, the real and
// imaginary parts of both modes are sums and differences of four real
// products,
//   sum cos(s a theta) cos(b theta),  sum sin(s a theta) sin(b theta),
//   sum sin(s a theta) cos(b theta),  sum cos(s a theta) sin(b theta),
// so all of them are one real matrix product over the particles, [cos, sin](s
// a theta) by [cos, sin](b theta): 2 multiply-adds per particle and mode on
// the FP64 matrix cores, and only about sqrt(M) phases per particle, against
// 6 operations of a rotation and two additions per particle and mode (and a
// fresh phase every 16 modes) on the vector pipe. A workgroup stages the
// phases of 64 particles at a time in LDS and four waves multiply them out
// (v_mfma_f64_16x16x4: 8 values of a by the cosines or sines of 16 values
// of b, four particles per instruction). Every phase table entry is at
// most 7 rotations from a phase reduced mod 1 exactly, evaluated from a
// table of 256 unit vectors and a short polynomial.
//   wide   (M > 112): s = 31, b <= 15; a workgroup holds 32 values of a (8
//          per wave), 976 modes and more by further mode blocks; a wave
//          whose tile of a is not needed takes a share of the particles.
//          Two teams of four waves work in opposite phases: while one
//          generates a group's phases (vector pipe), the other multiplies
//          its own (matrix pipe).
//   narrow (M <= 112): s = 15, b <= 7, 8 values of a: one tile holds every
//          mode, and each wave takes its own groups of 64 particles, with
//          no barrier between the waves. Up to four values of a (M <= 52) go
//          to v_mfma_f64_4x4x4 (four blocks of 4 x 4): once for the cosines and
//          once for the sines of a by the 16 columns, half the matrix time.
//   direct (small samples): a workgroup per 4, 8 or 16 modes, each thread a phase,
//          rotations and the sums of its particles, one exchange at the end: the
//          moments themselves, with no rows and no launch to sum them.
// The matrix instruction and the vector FMAs share a SIMD's FP64 units, so
// what bounds it is their sum: the products (2 operations per particle and
// mode) and the phases. Measured on MI355X against the kernel of rotations
// (6 operations per particle and mode and two phases every 16 modes): 65,536
// particles to order 911 in 10.2 us (47.6), 1,048,576 to order 46 in 18.8 us
// (49.0; 17.8 with the 4 x 4 blocks), to order 911 in 111 us (39 TFLOP/s; the
// products alone 76 us).
//
// Layout of the double instruction (one value per lane for A and B, four for
// C): lane l holds A[l % 16][l / 16], B[l / 16][l % 16] and, in element r,
// C[4 r + l / 16][l % 16]. Of the 4 x 4 one, with block b = l / 4 % 4: A_b[l %
// 4][l / 16], B_b[l / 16][l % 4], C_b[l / 16][l % 4].
#include <climits>
#include <cmath>

#include "dev_layout.hpp"
#include "kde_internal.hpp"

namespace kde {

using f64x4 = double __attribute__((ext_vector_type(4)));

constexpr double kFourierTail = 1e-18;  // rho_M below this ends the series
constexpr int kMomGroup = 64;           // particles whose phases are in LDS at a time (per wave when narrow)
constexpr int kMomPad = kMomGroup + 2;  // padded so that the 8 or 16 rows read together lie in different banks
constexpr int kWideStep = 31, kWideB = 16, kWideA = 32;  // mode block: a < 32
constexpr int kNarrowStep = 15, kNarrowB = 8, kNarrowA = 8;
constexpr int kNarrowMax = kNarrowStep * (kNarrowA - 1) + kNarrowB - 1;  // 112
constexpr int kMomBlock = 512;          // threads of a moment workgroup: two teams, or eight waves
constexpr int kMomTeam = 256;
constexpr int kMomWaves = kMomBlock / 64;
constexpr int64_t kMomChunks = 256;     // particle chunks a launch aims for (one workgroup per CU: its LDS)

// How the moments of n particles to order M are cut. The scans of a sample
// and the batched engine take the same plan (a function of n, M and the rows
// that the scan's workspace holds), so they sum the same partials in the same order.
struct MomentPlan {
  int M;
  int narrow, direct;    // direct: modes of a workgroup
  int mblocks;           // mode blocks
  int tiles, ks;         // wide: tiles of 8 a in a mode block, waves sharing a tile (each a share of the particles)
  int na;                // values of a (narrow)
  int64_t per;           // particles per chunk
  int64_t chunks, rows;  // rows of 2 M partial sums, one per chunk; a single one is the result
};

__host__ __device__ inline MomentPlan narrow_plan(int64_t n, int M, int64_t max_rows = kMomChunks) {
  MomentPlan p{};
  p.M = M;
  p.narrow = 1;
  p.mblocks = p.tiles = p.ks = 1;
  p.na = M <= kNarrowB - 1 ? 1 : (M - (kNarrowB - 1) + kNarrowStep - 1) / kNarrowStep + 1;
  p.per = kMomBlock * ceil_div(ceil_div(n, kMomBlock), max_rows < kMomChunks ? max_rows : kMomChunks);
  p.chunks = ceil_div(n, p.per);
  p.rows = p.chunks;
  return p;
}

// Tiles per mode block of the wide form: four, or fewer where the workspace holds
// too few rows to fill the chip with chunks (a workgroup with one tile takes about
// half the time per group of particles). Then the direct form, with the fewest
// modes per workgroup that leave one workgroup per CU, where its time is below
// the matrix forms' with their second launch, by the times of the parts in ns.
// Whole scans of 8 concentrations to 1e4, direct against matrix forms: 1000 to
// 8192 particles 18 us (21), 12,000 21.0 (21.0), 16,384 24.0 (20.5). With rows for
// 46 to 60 chunks in the pair layout and two or one tiles: 20,011 particles 20.9 us,
// 24.2 with four tiles and 20.9 with all 157 rows; a single concentration pays
// more (23.4 against 20.4), and kappas near 1e6, whose rows are 146 KB, most:
// 18,000 particles 95 us (52), 65,536 with one concentration 144 (99).
inline double wide_group_ns(int tiles) { return tiles >= 3 ? 850.0 : (tiles == 2 ? 600.0 : 450.0); }
inline double direct_particle_ns(int modes) { return modes == 4 ? 0.46 : (modes == 8 ? 0.65 : 1.1); }
constexpr double kNarrowGroupNs = 600.0, kSecondLaunchNs = 3000.0;

inline MomentPlan moment_plan(int64_t n, int M, int64_t max_rows) {
  MomentPlan p{};
  const int64_t most = max_rows > 1 ? max_rows : 1;
  double ns = 0.0;
  if (M <= kNarrowMax) {
    p = narrow_plan(n, M, most);
    ns = double(p.per / kMomBlock) * kNarrowGroupNs;
  } else {
    p.M = M;
    const int na = (M - (kWideB - 1) + kWideStep - 1) / kWideStep + 1;
    const int all = (na + 7) / 8;
    for (int tiles = all < 4 ? all : 4;; tiles = tiles == 3 ? 2 : tiles / 2) {
      p.tiles = tiles;
      p.ks = tiles == 1 ? 4 : (tiles == 2 ? 2 : 1);
      p.mblocks = (all + tiles - 1) / tiles;
      int64_t aim = kMomChunks / p.mblocks;
      if (aim > most) aim = most;
      if (aim < 1) aim = 1;
      p.per = 2 * kMomGroup * ceil_div(ceil_div(n, 2 * kMomGroup), aim);  // the teams take groups in turn
      p.chunks = ceil_div(n, p.per);
      const int finer = tiles == 3 ? 2 : tiles / 2;
      if (tiles == 1 || p.chunks * ((all + finer - 1) / finer) > kMomChunks || p.per == 2 * kMomGroup) break;
    }
    p.rows = p.chunks;
    ns = double(p.per / kMomGroup + 1) * wide_group_ns(p.tiles) * double(ceil_div(p.chunks * p.mblocks, kMomChunks));
  }
  int modes = 4;
  while (modes < 16 && ceil_div(M, modes) > kMomChunks) modes *= 2;
  const int64_t blocks = ceil_div(M, modes);
  const double direct_ns = double(n) * direct_particle_ns(modes) * double(ceil_div(blocks, kMomChunks));
  if (direct_ns >= ns + (p.rows > 1 ? kSecondLaunchNs : 0.0)) return p;
  p = MomentPlan{};
  p.M = M;
  p.direct = modes;
  p.mblocks = int(blocks);
  p.tiles = p.ks = 1;
  p.per = n;
  p.chunks = p.rows = 1;
  return p;
}

// Phase exp(i 2 pi m f) for f in [0, 1]: m f reduced mod 1 with its
// rounding error recovered, so the angle is exact to a few units of f's
// last place times m.
__device__ __forceinline__ void phase(int m, double f, double& c, double& s) {
  const double t = double(m) * f;
  const double e = fma(double(m), f, -t);
  const double fr = (t - floor(t)) + e;
  sincospi(2.0 * fr, &s, &c);
}

// Position as a fraction of the period: wrap_d(x, L) / L. For x inside [0, L)
// the quotient comes from the reciprocal and one correction (within a
// rounding unit of the division), elsewhere from the wrap.
__device__ __forceinline__ double period_fraction(double x, double L, double inv_L) {
  const double q0 = x * inv_L;
  const double q = fma(fma(-q0, L, x), inv_L, q0);
  return (q0 >= 0.0 && q0 < 1.0) ? q : wrap_d(x, L) / L;
}

// exp(i 2 pi j / 256), one entry per thread of the first kMomTeam.
__device__ __forceinline__ void unit_table_fill(double2* unit) {
  if (threadIdx.x < 256) {
    double s, c;
    sincospi(double(threadIdx.x) / 128.0, &s, &c);
    unit[threadIdx.x] = double2{c, s};
  }
}

// phase() from the table: m f = k / 256 + r mod 1, |r| <= 1/512 (and the
// product's rounding error), then exp(i 2 pi r) by its Taylor series (|2 pi
// r| <= 0.0123: the first terms left out are below 2e-20) times the table
// entry. Its error is about a rounding unit, absolute, like that of the
// rotations that follow; sincospi's relative accuracy near the axes is not
// needed in a sum.
__device__ __forceinline__ double2 table_phase(double m, double f, const double2* unit) {
  const double t = m * f;
  const double e = fma(m, f, -t);
  const double k = rint(t * 256.0);
  const double r = fma(k, -1.0 / 256.0, t) + e;
  const double2 u = unit[int(k) & 255];
  const double x = r * 6.283185307179586;
  const double x2 = x * x;
  const double cm = x2 * fma(x2, fma(x2, -1.0 / 720.0, 1.0 / 24.0), -0.5);  // cos - 1
  const double sn = x * fma(x2, fma(x2, fma(x2, -1.0 / 5040.0, 1.0 / 120.0), -1.0 / 6.0), 1.0);
  return double2{fma(u.x, cm, fma(-u.y, sn, u.x)), fma(u.y, cm, fma(u.x, sn, u.y))};
}
__device__ __forceinline__ double2 rotate(double2 z, double2 w) {
  return double2{fma(z.x, w.x, -(z.y * w.y)), fma(z.y, w.x, z.x * w.y)};
}

struct MomSmem {
  // narrow: 16 rows per wave; wide: 48 rows per team
  double2 z[kMomWaves * (kNarrowA + kNarrowB) * kMomPad];
  double2 unit[256];
};

// One (chunk, mode block) of the wide form, into the chunk's row of 2 M doubles. Every thread of the workgroup must call this.
template <typename T>
__device__ __forceinline__ void moments_wide(const T* __restrict__ x, int64_t lo, int64_t hi, double L,
                                             const MomentPlan& p, int mb, double* __restrict__ out, MomSmem& sm,
                                             uint32_t* status) {
  const int tid = threadIdx.x, lane = tid & 63, team = tid / kMomTeam, w = (tid % kMomTeam) >> 6;
  double2(*za)[kMomPad] = reinterpret_cast<double2(*)[kMomPad]>(sm.z) + team * (kWideA + kWideB);
  double2(*zb)[kMomPad] = za + kWideA;
  const int i16 = lane & 15, k4 = lane >> 4;
  const int tile = w % p.tiles, slice = w / p.tiles;  // slice < ks: this wave multiplies
  const int steps = (kMomGroup / 4) / p.ks;
  const int M = p.M;
  const double inv_L = 1.0 / L;
  // values of a this mode block needs, from a0 on
  const int a0 = 8 * p.tiles * mb;
  const int na = min((M - (kWideB - 1) + kWideStep - 1) / kWideStep + 1 - a0, 8 * p.tiles);
  const bool gen = 8 * w < na;  // wave w also generates the phases of a = a0 + 8 w ..
  const bool mul = slice < p.ks && 8 * tile < na;
  const double m_a = double(kWideStep * (a0 + 8 * w));
  f64x4 acc0 = {0.0, 0.0, 0.0, 0.0}, acc1 = {0.0, 0.0, 0.0, 0.0};
  const int groups = int((hi - lo + kMomGroup - 1) / kMomGroup);
  const double* arow = reinterpret_cast<const double*>(&za[8 * tile + (i16 & 7)][0]) + (i16 >> 3);
  const double2* brow = zb[i16];
  const int p0 = 4 * steps * slice + k4;
  int64_t j = lo + team * kMomGroup + lane;
  T xn = j < hi ? x[j] : T(0);
  // interval t: the team of t's parity generates group t, the other
  // multiplies group t - 1
  for (int t = 0; t <= groups; ++t) {
    if ((t & 1) == team) {
      if (t < groups) {
        const bool valid = j < hi;
        const double xv = double(xn);
        j += 2 * kMomGroup;
        xn = j < hi ? x[j] : T(0);  // this team's next group, in flight over this one's work
        if (mb == 0 && w == 0) note_numeric(status, !isfinite(xv), false);
        const double f = period_fraction(xv, L, inv_L);
        const double2 z1 = table_phase(1.0, f, sm.unit);
        double2 z = table_phase(double(4 * w), f, sm.unit);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          zb[4 * w + k][lane] = valid ? z : double2{0.0, 0.0};
          z = rotate(z, z1);
        }
        if (gen) {
          const double2 zs = table_phase(double(kWideStep), f, sm.unit);
          z = table_phase(m_a, f, sm.unit);
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            za[8 * w + k][lane] = z;
            z = rotate(z, zs);
          }
        }
      }
    } else if (t >= 1 && mul) {
      auto product = [&](auto count) {
        constexpr int kSteps = decltype(count)::value;
        double av[kSteps];
        double2 bv[kSteps];
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
          av[u] = arow[2 * (p0 + 4 * u)];
          bv[u] = brow[p0 + 4 * u];
        }
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
          acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u], bv[u].x, acc0, 0, 0, 0);
          acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u], bv[u].y, acc1, 0, 0, 0);
        }
      };
      if (p.ks == 1)
        product(std::integral_constant<int, kMomGroup / 4>{});
      else if (p.ks == 2)
        product(std::integral_constant<int, kMomGroup / 8>{});
      else
        product(std::integral_constant<int, kMomGroup / 16>{});
    }
    __syncthreads();
  }
  // a tile's sums: to the first wave's those of the others, the teams' and the
  // slices' in order
  double* red = reinterpret_cast<double*>(sm.z);
  const bool first = team == 0 && slice == 0;
  if (!first) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      red[r * kMomBlock + tid] = acc0[r];
      red[(4 + r) * kMomBlock + tid] = acc1[r];
    }
  }
  __syncthreads();
  if (first && mul) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      acc0[r] += red[r * kMomBlock + tid + kMomTeam];
      acc1[r] += red[(4 + r) * kMomBlock + tid + kMomTeam];
      for (int q = 1; q < p.ks; ++q) {
        const int at = tid + 64 * q * p.tiles;
        acc0[r] += red[r * kMomBlock + at] + red[r * kMomBlock + at + kMomTeam];
        acc1[r] += red[(4 + r) * kMomBlock + at] + red[(4 + r) * kMomBlock + at + kMomTeam];
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int a = a0 + 8 * tile + 4 * h + k4, b = i16;
      const double cc = acc0[h], sc = acc0[h + 2], cs = acc1[h], ss = acc1[h + 2];
      const int mp = kWideStep * a + b, mm = kWideStep * a - b;
      if (mp >= 1 && mp <= M) {
        out[2 * (mp - 1)] = cc - ss;
        out[2 * (mp - 1) + 1] = sc + cs;
      }
      if (a >= 1 && b >= 1 && mm <= M) {
        out[2 * (mm - 1)] = cc + ss;
        out[2 * (mm - 1) + 1] = sc - cs;
      }
    }
  }
  __syncthreads();
}

// One chunk of the narrow form; writes the chunk's row of 2 M doubles.
template <typename T>
__device__ __forceinline__ void moments_narrow(const T* __restrict__ x, int64_t lo, int64_t hi, double L,
                                               const MomentPlan& p, double* __restrict__ out, MomSmem& sm,
                                               uint32_t* status) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  double2(*za)[kMomPad] = reinterpret_cast<double2(*)[kMomPad]>(sm.z) + w * (kNarrowA + kNarrowB);
  double2(*zb)[kMomPad] = za + kNarrowA;
  const int i16 = lane & 15, k4 = lane >> 4;
  const double* arow = reinterpret_cast<const double*>(&za[i16 & 7][0]) + (i16 >> 3);
  const double* brow = reinterpret_cast<const double*>(&zb[i16 & 7][0]) + (i16 >> 3);
  const double inv_L = 1.0 / L;
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  int64_t j = lo + tid;
  T xn = j < hi ? x[j] : T(0);
  for (int64_t g = lo + 64 * w; g < hi; g += kMomBlock) {
    const bool valid = j < hi;
    const double xv = double(xn);
    j += kMomBlock;
    xn = j < hi ? x[j] : T(0);  // the next group's, in flight over this one's work
    note_numeric(status, !isfinite(xv), false);
    const double f = period_fraction(xv, L, inv_L);
    const double2 z1 = table_phase(1.0, f, sm.unit);
    const double2 zs = table_phase(double(kNarrowStep), f, sm.unit);
    double2 z = {1.0, 0.0};
#pragma unroll
    for (int k = 0; k < kNarrowB; ++k) {
      zb[k][lane] = valid ? z : double2{0.0, 0.0};
      z = k == 0 ? z1 : rotate(z, z1);
    }
    z = {1.0, 0.0};
    for (int k = 0; k < p.na; ++k) {
      za[k][lane] = z;
      z = rotate(z, zs);
    }
    // a wave's LDS accesses complete in order; the fences keep the compiler
    // from moving them across each other
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (p.na <= 4) {
      // four values of a fill half of the 16 x 16 tile's rows: the cosines
      // and the sines by four columns blocks each instead
#pragma unroll
      for (int t = 0; t < kMomGroup / 4; ++t) {
        const double2 av = za[lane & 3][4 * t + k4];
        const double bv = brow[2 * (4 * t + k4)];
        acc[0] = __builtin_amdgcn_mfma_f64_4x4x4f64(av.x, bv, acc[0], 0, 0, 0);
        acc[2] = __builtin_amdgcn_mfma_f64_4x4x4f64(av.y, bv, acc[2], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int t = 0; t < kMomGroup / 4; ++t)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(arow[2 * (4 * t + k4)], brow[2 * (4 * t + k4)], acc, 0, 0, 0);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  // the waves' sums in wave order, then the modes from the products
  double* red = reinterpret_cast<double*>(sm.z);  // the phases are no longer needed
#pragma unroll
  for (int r = 0; r < 4; ++r) red[(w * 64 + lane) * 4 + r] = acc[r];
  __syncthreads();
  if (w == 0) {
    double v[4], u[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      v[r] = 0.0;
      for (int q = 0; q < kMomWaves; ++q) v[r] += red[(q * 64 + lane) * 4 + r];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) u[r] = __shfl_xor(v[r], 8, 64);  // the sines' columns
    const int b = i16;
    if (b < kNarrowB) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int a = 4 * h + k4;
        const double cc = v[h], sc = v[h + 2], cs = u[h], ss = u[h + 2];
        const int mp = kNarrowStep * a + b, mm = kNarrowStep * a - b;
        if (a < p.na && mp >= 1 && mp <= p.M) {
          out[2 * (mp - 1)] = cc - ss;
          out[2 * (mp - 1) + 1] = sc + cs;
        }
        if (a < p.na && a >= 1 && b >= 1 && mm <= p.M) {
          out[2 * (mm - 1)] = cc + ss;
          out[2 * (mm - 1) + 1] = sc - cs;
        }
      }
    }
  }
  __syncthreads();
}

// K modes of the direct form, over all particles, into the moments `out`.
template <int K, typename T>
__device__ __forceinline__ void moments_direct(const T* __restrict__ x, int64_t n, double L, int M, int mb,
                                               double* __restrict__ out, MomSmem& sm, uint32_t* status) {
  constexpr int kVals = 2 * K;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int m0 = 1 + K * mb;
  const double inv_L = 1.0 / L;
  double v[kVals];
#pragma unroll
  for (int k = 0; k < kVals; ++k) v[k] = 0.0;
#pragma unroll 2
  for (int64_t j = tid; j < n; j += kMomBlock) {
    const double xv = double(x[j]);
    if (mb == 0) note_numeric(status, !isfinite(xv), false);
    const double f = period_fraction(xv, L, inv_L);
    const double2 z1 = table_phase(1.0, f, sm.unit);
    double2 z;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      z = k % 8 == 0 ? table_phase(double(m0 + k), f, sm.unit) : rotate(z, z1);
      v[2 * k] += z.x;
      v[2 * k + 1] += z.y;
    }
  }
  // the lanes' sums in a tree over all values at once: after the exchange at
  // distance d a lane keeps the half of the values that its bit d names
  int half = K, d = 32;
#pragma unroll
  for (; half >= 1; half >>= 1, d >>= 1) {
    const bool up = (lane & d) != 0;
#pragma unroll
    for (int k = 0; k < half; ++k) {
      const double keep = up ? v[k + half] : v[k];
      const double give = up ? v[k] : v[k + half];
      v[k] = keep + shfl_xor_d(give, d);
    }
  }
#pragma unroll
  for (; d >= 1; d >>= 1) v[0] += shfl_xor_d(v[0], d);
  constexpr int kSame = 64 / kVals;  // lanes that hold one value
  double* red = reinterpret_cast<double*>(sm.z);
  if (lane % kSame == 0) red[w * kVals + lane / kSame] = v[0];
  __syncthreads();
  if (tid < kVals) {
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < kMomWaves; ++q) t += red[q * kVals + tid];
    if (m0 + (tid >> 1) <= M) out[2 * (m0 - 1) + tid] = t;
  }
  __syncthreads();
}

// Unit (chunk, mode block) of a set's moments into its partial rows, by a
// workgroup of kMomBlock threads; sm.unit must be filled and visible.
template <typename T>
__device__ __forceinline__ void moments_unit(const T* __restrict__ x, int64_t n, double L, const MomentPlan& p,
                                             int64_t chunk, int mb, double* __restrict__ partials, MomSmem& sm,
                                             uint32_t* status) {
  const int64_t lo = chunk * p.per, hi = min(n, lo + p.per);
  if (p.direct == 4)
    moments_direct<4>(x, n, L, p.M, mb, partials, sm, status);
  else if (p.direct == 8)
    moments_direct<8>(x, n, L, p.M, mb, partials, sm, status);
  else if (p.direct == 16)
    moments_direct<16>(x, n, L, p.M, mb, partials, sm, status);
  else if (p.narrow)
    moments_narrow(x, lo, hi, L, p, partials + chunk * 2 * int64_t(p.M), sm, status);
  else
    moments_wide(x, lo, hi, L, p, mb, partials + chunk * 2 * int64_t(p.M), sm, status);
}

// Sum of the partial rows, kRedCols columns per workgroup: thread (y, c)
// adds rows y, y + 16, ... in order, then the 16 partial sums are added in
// a tree. (Rows read by 16 threads side by side: the serial chain of a
// column is rows / 16 additions.)
constexpr int kRedCols = 16;

__device__ __forceinline__ void moments_reduce(const double* __restrict__ partials, int64_t rows, int cols, int64_t cb,
                                               double* __restrict__ S, double* red) {
  const int c = threadIdx.x % kRedCols, y = threadIdx.x / kRedCols;
  constexpr int ny = kBlock / kRedCols;
  const int64_t col = cb * kRedCols + c;
  double v = 0.0;
  if (col < cols) {
#pragma unroll 4
    for (int64_t r = y; r < rows; r += ny) v += partials[r * cols + col];
  }
  red[threadIdx.x] = v;
  __syncthreads();
  if (y == 0 && col < cols) {
    double t[ny];
#pragma unroll
    for (int q = 0; q < ny; ++q) t[q] = red[q * kRedCols + c];
#pragma unroll
    for (int d = ny / 2; d >= 1; d /= 2)
#pragma unroll
      for (int q = 0; q < d; ++q) t[q] += t[q + d];
    S[col] = t[0];
  }
  __syncthreads();
}

// -------------------------------------------------------------- the series

// a b rescaled by a power of two (exact) so that products of many of these
// non-negative matrices stay in range.
struct Mat2 {
  double a, b, c, d;
};
__device__ __forceinline__ Mat2 mat_norm(const Mat2& m) {
  const double mx = fmax(fmax(m.a, m.b), fmax(m.c, m.d));
  const int e = __builtin_amdgcn_frexp_exp(mx);  // 0 for zero
  return Mat2{ldexp(m.a, -e), ldexp(m.b, -e), ldexp(m.c, -e), ldexp(m.d, -e)};
}
__device__ __forceinline__ Mat2 mat_mul(const Mat2& x, const Mat2& y) {
  return mat_norm(Mat2{fma(x.a, y.a, x.b * y.c), fma(x.a, y.b, x.b * y.d), fma(x.c, y.a, x.d * y.c),
                       fma(x.c, y.b, x.d * y.d)});
}

// Static LDS of the series of one concentration; its dynamic part is 2 (M +
// 1) doubles (series_lds): the ratios, then |S_m|^2.
struct ScanSmem {
  Mat2 tot[kBlock / 64];
  double ptot[kBlock / 64];
  double red[kBlock / 64][3];
};
// Where the backward recurrence of a series to order M starts, and the doubles
// that hold its values (from index 1) over a bracket that ends at kappa: the
// refinement evaluates the end at exp(log(kappa)), which can exceed kappa by
// a rounding unit, and where M^2 + 40 kappa is a perfect square the series
// is one longer then.
__host__ __device__ inline int series_length(int M, double kappa) {
  return int(ceil(sqrt(double(M) * double(M) + 40.0 * kappa))) + 16;
}
__host__ __device__ inline int series_slots(int M, double kappa) { return series_length(M, kappa) + 2; }
__host__ __device__ inline size_t series_lds(int M) { return size_t(2) * size_t(M + 1) * sizeof(double); }

// The ratios r_m = I_m/I_{m-1} (m = 1..M) of one concentration into LDS by
// the whole workgroup. Thread t owns the run m = lo..hm and gets p, the
// product of the ratios before it (so that rho_m = p r_lo .. r_m). Ends with a
// barrier.
//
// The backward recurrence r_m = kappa / (2m + kappa r_{m+1}), started at
// r_{Ms+1} = 0, applies the Mobius maps with matrices [[0, kappa], [kappa,
// 2m]] to the vector (0, 1). Each thread composes the maps of its run of
// consecutive m (non-negative matrices rescaled by powers of two: no
// cancellation); a suffix product over the workgroup, by shuffles inside a
// wave and one exchange between the waves, gives every run the vector
// entering it; each thread walks its run on that vector (so the divisions do
// not wait for each other); a prefix product follows. The composition is a
// reassociation of the recurrence; its rounding grows with the depth of the
// tree and not with the length of the chain.
__device__ __forceinline__ void series_ratios(double kappa, int M, double* __restrict__ ratio, ScanSmem& sm, int& lo,
                                              int& hm, double& p) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  constexpr int kWaves = kBlock / 64;
  const int Ms = series_length(M, kappa);
  const int len = (Ms + kBlock - 1) / kBlock;
  lo = 1 + t * len;
  const int hi = min(Ms, (t + 1) * len);  // empty when lo > hi
  Mat2 P{1.0, 0.0, 0.0, 1.0};
  for (int m = hi; m >= lo; --m) {
    const double m2 = 2.0 * double(m);
    P = mat_norm(Mat2{kappa * P.c, kappa * P.d, fma(kappa, P.a, m2 * P.c), fma(kappa, P.b, m2 * P.d)});
  }
  // inclusive suffix products inside the wave
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const Mat2 o{__shfl_down(P.a, d, 64), __shfl_down(P.b, d, 64), __shfl_down(P.c, d, 64), __shfl_down(P.d, d, 64)};
    const Mat2 q = mat_mul(P, o);
    if (lane + d < 64) P = q;
  }
  if (lane == 0) sm.tot[w] = P;
  __syncthreads();
  // the vector entering this wave from the waves above, then this thread
  double vx = 0.0, vy = 1.0;
  for (int k = kWaves - 1; k > w; --k) {
    const Mat2 T = sm.tot[k];
    const double nx = fma(T.a, vx, T.b * vy), ny = fma(T.c, vx, T.d * vy);
    const int e = __builtin_amdgcn_frexp_exp(fmax(nx, ny));
    vx = ldexp(nx, -e);
    vy = ldexp(ny, -e);
  }
  {
    const Mat2 o{__shfl_down(P.a, 1, 64), __shfl_down(P.b, 1, 64), __shfl_down(P.c, 1, 64), __shfl_down(P.d, 1, 64)};
    if (lane < 63) {
      const double nx = fma(o.a, vx, o.b * vy), ny = fma(o.c, vx, o.d * vy);
      vx = nx;
      vy = ny;
    }
  }
  double sp = 1.0;
  for (int m = hi; m >= lo; --m) {
    // (x, y) <- (kappa y, kappa x + 2m y), r_m = x / y; rescaled so that y ~ 1
    const double nx = kappa * vy, ny = fma(kappa, vx, 2.0 * double(m) * vy);
    const int e = __builtin_amdgcn_frexp_exp(ny);
    vx = ldexp(nx, -e);
    vy = ldexp(ny, -e);
    if (m <= M) {
      const double r = vx / vy;
      ratio[m] = r;
      sp *= r;
    }
  }
  // exclusive prefix products of the runs' products
  double pp = sp;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const double o = __shfl_up(pp, d, 64);
    if (lane >= d) pp *= o;
  }
  if (lane == 63) sm.ptot[w] = pp;
  __syncthreads();  // also: every ratio is in LDS
  p = __shfl_up(pp, 1, 64);
  if (lane == 0) p = 1.0;
  for (int k = 0; k < w; ++k) p *= sm.ptot[k];
  hm = min(hi, M);
}

// rho_m (m = 1..M) of one concentration into LDS; ends with a barrier.
__device__ __forceinline__ void series_rho(double kappa, int M, double* __restrict__ rho, ScanSmem& sm) {
  int lo, hm;
  double p;
  series_ratios(kappa, M, rho, sm, lo, hm, p);
  for (int m = lo; m <= hm; ++m) {
    p *= rho[m];
    rho[m] = p;
  }
  __syncthreads();
}

// The same to a rounding unit, for series of at most kBlock modes (a thread's run
// is one). The composed maps leave a few units in a ratio, and a grid's nodes hang on
// single modes; they are taken out to first order: with r_m = (1 + d_m) times the exact
// ratio, the recurrence's residual e_m = r_m (2m + kappa r_{m+1}) - kappa, evaluated with
// its products' and sum's remainders, gives d_m = e_m / kappa - r_m r_{m+1} d_{m+1},
// an affine recurrence solved by a suffix scan, and rho_m is divided by the
// product of its ratios' 1 + d.
__device__ __forceinline__ void series_rho_exact(double kappa, int M, double* __restrict__ rho, ScanSmem& sm) {
  int m, hm;
  double p;
  series_ratios(kappa, M, rho, sm, m, hm, p);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const double r = m <= M ? rho[m] : 0.0;
  double a = 0.0, b = 0.0;  // d_m = a + b d_{m+1}
  if (m < M && kappa > 0.0) {
#pragma clang fp contract(off)
    const double r1 = rho[m + 1], m2 = 2.0 * double(m);
    const double h = kappa * r1, s = m2 + h, bb = s - m2;
    const double sl = ((m2 - (s - bb)) + (h - bb)) + fma(kappa, r1, -h);
    const double q = r * s;
    a = ((q - kappa) + fma(r, sl, fma(r, s, -q))) / kappa;
    b = -r * r1;
  }
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const double oa = __shfl_down(a, d, 64), ob = __shfl_down(b, d, 64);
    if (lane + d < 64) {
      a = fma(b, oa, a);
      b *= ob;
    }
  }
  if (lane == 0) {
    sm.red[w][0] = a;
    sm.red[w][1] = b;
  }
  __syncthreads();  // also: every ratio has been read
  double above = 0.0;
  for (int k = kBlock / 64 - 1; k > w; --k) above = fma(sm.red[k][1], above, sm.red[k][0]);
  double d = fma(b, above, a);
#pragma unroll
  for (int k = 1; k < 64; k <<= 1) {
    const double o = __shfl_up(d, k, 64);
    if (lane >= k) d += o;
  }
  if (lane == 63) sm.red[w][2] = d;
  __syncthreads();
  for (int k = 0; k < w; ++k) d += sm.red[k][2];
  if (m <= M) rho[m] = fma(-d, p * r, p * r);
  __syncthreads();
}

// A = sum_m rho_m^2 P_m, A0 = sum_m rho_m^2 (P_m - n), C = sum_m rho_m (P_m -
// n), m = 1..M, P_m = |S_m|^2, for one concentration, by the whole workgroup.
__device__ __forceinline__ void series_sums(double kappa, int M, const double* __restrict__ S, double n,
                                            double* __restrict__ dyn, ScanSmem& sm, double& A, double& A0, double& C) {
  double* ratio = dyn;
  double* pw = dyn + (M + 1);
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  for (int m = 1 + t; m <= M; m += kBlock) {
    const double sr = S[2 * (m - 1)], si = S[2 * (m - 1) + 1];
    pw[m] = fma(sr, sr, si * si);
  }
  int lo, hm;
  double p;
  series_ratios(kappa, M, ratio, sm, lo, hm, p);
  double a = 0.0, a0 = 0.0, c = 0.0;
  for (int m = lo; m <= hm; ++m) {
    p *= ratio[m];
    const double Pm = pw[m], q = Pm - n, p2 = p * p;
    a = fma(p2, Pm, a);
    a0 = fma(p2, q, a0);
    c = fma(p, q, c);
  }
  a = wave_sum(a);
  a0 = wave_sum(a0);
  c = wave_sum(c);
  if (lane == 0) {
    sm.red[w][0] = a;
    sm.red[w][1] = a0;
    sm.red[w][2] = c;
  }
  __syncthreads();
  A = A0 = C = 0.0;
#pragma unroll
  for (int k = 0; k < kBlock / 64; ++k) {
    A += sm.red[k][0];
    A0 += sm.red[k][1];
    C += sm.red[k][2];
  }
  __syncthreads();
}

// The objective and the pair sums of one concentration from the series.
__device__ __forceinline__ double cv_of_series(double A, double C, double n, double L) {
  return (2.0 * A / (n * n) - 4.0 * C / (n * (n - 1.0)) - 1.0) / L;
}
__device__ __forceinline__ double pair_sum_of_series(double D, double n, double L) {
  return (n * n - n + 2.0 * D) / (2.0 * L);
}

__device__ __forceinline__ int first_min(const double* v, int B) {
  int best = 0;
  for (int t = 1; t < B; ++t)
    if (v[t] < v[best]) best = t;
  return best;
}

struct SeriesSmem {
  ScanSmem scan;
  double v[KDE_MAX_KAPPAS];
  int last;
};

// Concentration b of the first B of a list of Ball, by one workgroup: its
// objective and pair sums (sums may be NULL). With `done`, a counter that
// starts at 0, the workgroup that finishes last (of B) finds the first
// minimum of cv[0..B) and returns its index in every thread; otherwise -1.
// Which workgroup that is changes nothing: the values are fixed.
__device__ __forceinline__ int series_unit(double kappa, int M, const double* __restrict__ S, double n, double L, int b,
                                           int B, int Ball, double* cv, double* __restrict__ sums,
                                           unsigned int* done, double* dyn, SeriesSmem& sm) {
  double A, A0, C;
  series_sums(kappa, M, S, n, dyn, sm.scan, A, A0, C);
  if (threadIdx.x == 0) {
    __hip_atomic_store(&cv[b], cv_of_series(A, C, n, L), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (sums) {
      sums[b] = pair_sum_of_series(A0, n, L);
      sums[Ball + b] = pair_sum_of_series(C, n, L);
    }
    if (done) {
      __threadfence();
      sm.last = atomicAdd(done, 1u) == unsigned(B - 1) ? 1 : 0;
    }
  }
  if (!done) return -1;
  __syncthreads();
  if (!sm.last) return -1;
  __threadfence();
  if (threadIdx.x < B)
    sm.v[threadIdx.x] = __hip_atomic_load(&cv[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  return first_min(sm.v, B);
}

// ---------------------------------------------- a grid density from moments

// rho[g] = (1/L)(1 + (2/n) sum_m rho_m Re(conj(S_m) e^{i m theta_g})), the
// deposit of n particles with one concentration, 256 nodes by one workgroup: `tab`
// (LDS) holds exp(i 2 pi k / Mg), k < Mg. Returns whether the result is as
// accurate as the sum over the particles: what is left of its rounding is about
// half a unit of the series' magnitude A = 1 + (2/n) sum_m rho_m |S_m|, so every node
// has to be at least A / 8 (a density with empty stretches fails this, and so
// does a NaN). Against long double, 131,072 particles on 256 nodes, the largest
// error of a node over 12 samples each (the sum over the particles: 5e-16 to
// 7e-16): 1 + a cos at kappa = 26 4.2e-16 for a = 0.5 and 5.8e-16 for a = 0.75
// (A / 6.7), at kappa = 144 3.4e-16 and 5.4e-16 (A / 7.3); a quarter in a clump of 0.02
// L at kappa = 144 (A / 6.8) 5.2e-16 (1.3e-15). Summed upwards from the first mode,
// without remainders and with coefficients of a few units it was 1.2e-15 to 4.3e-15.
constexpr double kSynthLow = 0.125;
constexpr int kSynthExact = 16;  // leading modes summed with their remainders
struct SynthSmem {
  double2 w[kNarrowMax + 1];
  double2 rest[kSynthExact + 1];  // what rounding takes from the first w
  double red[kBlock / 64][2];
};

// s += x, with what rounding takes added to `lost` (Knuth's two-sum).
__device__ __forceinline__ void add_exact(double& s, double x, double& lost) {
#pragma clang fp contract(off)
  const double t = s + x, b = t - s;
  lost += (s - (t - b)) + (x - b);
  s = t;
}

// Where the moments of a deposit lie: S, rho behind it (narrow_sums).
constexpr int kNarrowSums = 3 * kNarrowMax + 1;
struct NarrowSmem {
  ScanSmem scan;
  double rho[kNarrowMax + 1];
  double red[kBlock];
};
// Units of the launch that adds a deposit's partial rows: the column blocks, and one
// that makes rho_m meanwhile.
__host__ __device__ inline int narrow_units(int M) { return (2 * M + kRedCols - 1) / kRedCols + 1; }
__device__ __forceinline__ void narrow_sums(const double* __restrict__ partials, int64_t rows, int M, int unit,
                                            double kappa, double* __restrict__ S, unsigned int* ok,
                                            NarrowSmem& sm) {
  if (unit == 0 && threadIdx.x == 0) *ok = 1u;  // until a part of the synthesis refuses
  if (unit + 1 < narrow_units(M)) {
    moments_reduce(partials, rows, 2 * M, unit, S, sm.red);
  } else {
    series_rho_exact(kappa, M, sm.rho, sm.scan);
    for (int m = 1 + threadIdx.x; m <= M; m += kBlock) S[2 * kNarrowMax + m] = sm.rho[m];
  }
}

// Workgroups of it: a node per thread.
__host__ __device__ inline int synthesis_parts(int Mg) { return (Mg + kBlock - 1) / kBlock; }

__device__ __forceinline__ bool deposit_synthesis(int M, const double* __restrict__ S, double n, double L, int Mg,
                                                  int part, double* __restrict__ out, double2* __restrict__ tab,
                                                  SynthSmem& sm) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  for (int k = t; k < Mg; k += kBlock) {
    double sn, cs;
    sincospi(2.0 * double(k) / double(Mg), &sn, &cs);
    tab[k] = double2{cs, sn};
  }
  const double* rho = S + 2 * kNarrowMax;
  double mag = 0.0;
  for (int m = 1 + t; m <= M; m += kBlock) {
    const double2 s = {S[2 * (m - 1)], S[2 * (m - 1) + 1]}, w = {rho[m] * s.x, rho[m] * s.y};
    sm.w[m] = w;
    if (m <= kSynthExact)
      sm.rest[m] = {fma(rho[m], s.x, -w.x), fma(rho[m], s.y, -w.y)};
    mag += sqrt(fma(w.x, w.x, w.y * w.y));
  }
  __syncthreads();
  double low = INFINITY;
  const int g = part * kBlock + t;
  if (g < Mg) {
    // from the last mode, the smallest, down; the leading modes, whose sum is at
    // its full size, with the remainders of their products and sums
    double v = 0.0, vl = 0.0;
    int idx = int((unsigned(M) * unsigned(g)) % unsigned(Mg));
    auto next = [&]() {
      const double2 e = tab[idx];
      idx -= g;
      idx += idx < 0 ? Mg : 0;
      return e;
    };
    int m = M;
#pragma unroll 4
    for (; m > kSynthExact; --m) {
      const double2 e = next(), w = sm.w[m];
      v = fma(w.x, e.x, v);
      v = fma(w.y, e.y, v);
    }
#pragma unroll 4
    for (; m >= 1; --m) {
      const double2 e = next(), w = sm.w[m], r = sm.rest[m];
      const double px = w.x * e.x, py = w.y * e.y;
      vl += fma(w.x, e.x, -px) + fma(w.y, e.y, -py) + fma(r.x, e.x, r.y * e.y);
      add_exact(v, px, vl);
      add_exact(v, py, vl);
    }
    const double q = 2.0 * v / n;
    double d = 1.0, dl = (fma(-q, n, 2.0 * v) + 2.0 * vl) / n;
    add_exact(d, q, dl);
    d += dl;
    out[g] = d / L;
    low = d < INFINITY ? d : -1.0;  // (no number: refused)
  }
  mag = wave_sum(mag);
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    low = fmin(low, shfl_xor_d(low, m));
  }
  if (lane == 0) {
    sm.red[wv][0] = mag;
    sm.red[wv][1] = low;
  }
  __syncthreads();
  mag = 0.0;
#pragma unroll
  for (int k = 0; k < kBlock / 64; ++k) {
    mag += sm.red[k][0];
    low = fmin(low, sm.red[k][1]);
  }
  __syncthreads();
  return low >= kSynthLow * (1.0 + 2.0 * mag / n);  // false where a moment is no number: mag is none then
}

// -------------------------------------------------------------------- host

// Whether the deposit of n particles on Mg nodes with one concentration tries
// the moments first (double form; a concentration whose series fits the
// narrow form, kappa up to about 144.8): they cost about 20 us with the launches
// that find nothing to do, and 8 ps per particle beyond that, against 0.65 ps
// per particle and node (1,048,576 on 256 nodes: 28 us against 178; 131,072: 21
// and 36; 8192 on 4096: 22 and 104). Where the grid is refused, which the host
// cannot see, they come on top of the sum over the particles (200 us, and 46), so
// the line is drawn at 2^25 pairs, the second of these sizes.
__host__ __device__ inline bool deposit_tries_moments(int prec, int64_t n, int Mg) {
  return prec == KDE_F64 && n * int64_t(Mg) >= (int64_t(1) << 25);
}

// Order at which the series of a concentration is cut: the smallest m with
//   m asinh(m/k) - (sqrt(m^2 + k^2) - k) >= -log(kFourierTail),
// from where on rho_m < kFourierTail: Amos's bounds I_nu(k) / I_{nu-1}(k) <=
// k / (t + sqrt(t^2 + k^2)) = exp(-asinh(t/k)), t = nu - 1/2, give -log rho_m
// >= the sum of asinh((nu - 1/2)/k) over nu <= m, and the midpoint sum of the
// concave asinh is at least its integral over [0, m], the left-hand side.
// Newton's method from above (the left-hand side is convex). rho_m grows
// with kappa, so the order of the largest concentration serves a whole list.
// The root is taken where it is a number that an int holds: below
// kOrderKappaMin (rho_1 < kappa / 2) the order is 1, and no series is evaluated
// above KDE_MAX_FOURIER_KAPPA, whose concentrations get the order INT_MAX,
// longer than anything a caller compares it with (from 5.8e16 on the root
// exceeds an int, from 1e34 it is NaN).
inline double fourier_root(double k) {
  static const double lim = -std::log(kFourierTail);
  double m = std::sqrt(2.0 * lim * k) + 12.0;
  for (int it = 0; it < 4; ++it) {
    const double u = m / k, as = std::log(u + std::sqrt(u * u + 1.0));
    m -= (m * as - m * m / (std::sqrt(m * m + k * k) + k) - lim) / as;
  }
  return m;
}
constexpr double kOrderKappaMin = 1e-100;
inline int fourier_order(double k) {
  if (!(k > kOrderKappaMin)) return 1;
  if (k > KDE_MAX_FOURIER_KAPPA) return INT_MAX;
  const int m = int(std::ceil(fourier_root(k)));
  return m < 1 ? 1 : m;
}

// Concentrations with their series orders (fourier_order of each; the
// order grows with kappa, so a bracket's upper end bounds it inside).
struct FKappas {
  double k[KDE_MAX_KAPPAS];
  int order[KDE_MAX_KAPPAS];
};
inline FKappas fourier_list(const double* k, int B) {
  FKappas f{};
  for (int b = 0; b < B; ++b) {
    f.k[b] = k[b];
    f.order[b] = fourier_order(k[b]);
  }
  return f;
}

// Largest concentration whose CV terms for n particles are taken through the
// moments in the double form; larger ones are summed over pairs. The moments
// give the double sums with the diagonal in, so S1 and S2 carry a few
// rounding units of n K(0) (the pair kernel sums positive terms and carries
// none). Positions have n gaps to their next neighbours, L / n on average,
// and a kernel is down to exp(-1/2) at its width s = L / (2 pi sqrt(kappa));
// with a mean gap of at most s / 1.5 the n neighbouring pairs alone therefore
// give S2 >= 0.4 n K(0) wherever the particles lie (the even spacing gives
// exp(-1/4.5)), and more pairs only add to it. So n K(0) <= 2.6 S2, and the few
// units of it are a few units of S2; S1's kernel is wider. Against direct
// sums in double, over even, jittered, paired, random and clustered
// positions of 8 to 1000 particles at this bound: objective within 2e-15,
// pair sums within 1e-15. The route costs n x order multiply-adds against
// n^2 / 2 pair terms of 33 operations, so where the accuracy allows it, it is
// the faster one at every size measured (calls of 8 concentrations to 1e3 at
// n = 4096: 18 us against 381; of 32 to 1e4 at 65,536: 24 us against 44,000).
// The float form keeps its float pair terms: its results are those of float
// arithmetic, which the moments (in double) do not reproduce.
inline double scan_kappa_limit(int64_t n) {
  const double k = double(n) / (3.0 * 3.141592653589793);
  return std::fmin(k * k, KDE_MAX_FOURIER_KAPPA);
}
// How many leading concentrations of an ascending list are taken through the
// moments: those, but none of a sample within one tile whose list needs the pair
// kernel as well and would be spared too little of it: passes of four, each
// about as long as the sample, against two launches of about 9 us. 64
// particles, 8 concentrations to 1e4, three of them below the limit (no pass):
// 103 us over pairs alone, 109 by both; 30, 16 to 1e4, four below (one): 66 and
// 74; 200, 16 to 1e4, ten below (two): 305 and 199.
inline int scan_fourier_count(int prec, int64_t n, const double* kappas, int B) {
  if (prec != KDE_F64) return 0;
  const double lim = scan_kappa_limit(n);
  int b = 0;
  while (b < B && kappas[b] <= lim) ++b;
  const int spared = (B + 3) / 4 - (B - b + 3) / 4;
  if (b < B && n <= kCvTile && n * spared < 64) return 0;
  return b;
}

// The moments' part of a workspace: partial rows (where there is more than
// one), the moments, and a counter of the series.
struct ScanBufs {
  MomentPlan plan;
  double* partials;
  double* S;
  unsigned int* done;  // workgroups of the series that have written their value
};
// To order M, of n particles, in `room` bytes, which have to hold one row.
inline ScanBufs carve_scan(Carver& c, size_t room, int64_t n, int M) {
  ScanBufs b{};
  b.done = c.take<unsigned int>(1);
  b.S = c.take<double>(size_t(2) * size_t(M));
  const size_t before = round_up(c.used, 256), row = size_t(2) * size_t(M) * sizeof(double);
  b.plan = moment_plan(n, M, before < room ? int64_t((room - before) / row) : 0);
  b.partials = b.plan.rows > 1 ? c.take<double>(size_t(b.plan.rows) * 2 * size_t(M)) : b.S;
  return b;
}

// Moments of x into b.S (fourier.hip). The launches record t0 as their
// start, `done` is zeroed. launch_moment_rows stops at the partial rows.
template <typename T>
kde_status launch_moment_rows(const T* x, int64_t n, double L, const ScanBufs& b, hipStream_t s, hipEvent_t t0,
                              hipEvent_t t1, uint32_t* status);
template <typename T>
kde_status launch_moments(const T* x, int64_t n, double L, const ScanBufs& b, hipStream_t s, hipEvent_t t0,
                          hipEvent_t t1, uint32_t* status);
// The series of concentrations [0, B) of a list of Ball: cv[b], sums[b],
// sums[Ball + b] (sums may be NULL), and the first minimum into *argmin when
// it is not NULL.
kde_status launch_series(const ScanBufs& b, int M, int64_t n, double L, const FKappas& kap, int B, int Ball,
                         double* cv, double* sums, int32_t* argmin, hipStream_t s, hipEvent_t t1);

}  // namespace kde
