// Grid density, field gather and adaptive widths with von Mises kernels.
//
// Deposit (Sec. II.B Eq. kde; Sec. II.C step 3 for per-particle widths):
//   rho[g] = (1/N) sum_i w_i exp(-2 kappa_i s_ig^2),
//   s_ig = sin(pi (x_g - x_i) / L),  w_i = 1 / (L I0e(kappa_i)).
// The grid is small (M <= 4096) and every particle touches every node, so
// a workgroup owns the whole grid for one contiguous chunk of particles:
// the chunk is staged in LDS (half-angle vector, exponent scale, weight)
// and read by all lanes at the same address (broadcast), each thread
// accumulating its own node(s). Per-chunk grids go to fixed slots and are
// summed in a fixed order. The cost is one exponential per (particle, node):
// transcendental-bound, not HBM-bound, at every grid size used here.
//
// Gather (field interpolation of Sec. III.A with the same kernels):
//   out[i] = (L/M) w_i sum_g F_g exp(-2 kappa_i s_ig^2),
// one thread per particle with the node table in LDS.
//
// Adaptive widths (Sec. II.C, Eq. adaptive_width): the pilot grid is
// interpolated linearly at each particle, its logarithms are averaged in
// double (fixed-order reduction), and kappa_i = kappa* exp(2 alpha (log f_i
// - log g)) is written per particle.
//
// The first-order (triangular) shape of adjustable width (dev_tri.hpp)
// deposits and gathers with the same decomposition; its per-particle
// parameter is the half-width h_i. Adaptive widths are von Mises only.
#include "dev_density.hpp"
#include "dev_fourier.hpp"
#include "dev_tri.hpp"

namespace kde {

// Dynamic LDS: the node table, M SinCos<T> (2 M values of T).
template <typename T, bool PER, int G>
__global__ void __launch_bounds__(kBlock) deposit_kernel(const T* __restrict__ x, const T* __restrict__ kap,
                                                        double kappa_g, int64_t n, int M, double L, int chunk,
                                                        double* __restrict__ partials, uint32_t* status,
                                                        const unsigned int* skip) {
  __shared__ DepSmem<T> sm;
  if (skip && *skip) return;  // the moments gave the grid
  extern __shared__ __align__(16) unsigned char dyn[];
  SinCos<T>* tab = reinterpret_cast<SinCos<T>*>(dyn);
  deposit_table(n, M, tab);
  const int64_t lo = int64_t(blockIdx.x) * chunk;
  const int cnt = int(min(int64_t(chunk), n - lo));
  deposit_block<T, PER, G>(x, kap, kappa_g, n, M, L, lo, cnt, partials + int64_t(blockIdx.x) * M, tab, sm, status);
}

// The grid from the particles' moments (dev_fourier.hpp); *ok becomes 0 where
// the sum over the particles has to follow. Dynamic LDS: Mg unit vectors.
__global__ void __launch_bounds__(kBlock) deposit_synthesis_kernel(const double* __restrict__ S, int M, double n,
                                                                  double L, int Mg, double* __restrict__ rho,
                                                                  unsigned int* ok) {
  __shared__ SynthSmem sm;
  extern __shared__ __align__(16) unsigned char dyn[];
  const bool good = deposit_synthesis(M, S, n, L, Mg, blockIdx.x, rho, reinterpret_cast<double2*>(dyn), sm);
  if (!good && threadIdx.x == 0) *ok = 0u;
}

// The rows' sums and the series' coefficients for it.
__global__ void __launch_bounds__(kBlock) deposit_sums_kernel(const double* __restrict__ partials, int64_t rows, int M,
                                                             double kappa, double* __restrict__ S,
                                                             unsigned int* ok) {
  __shared__ NarrowSmem sm;
  narrow_sums(partials, rows, M, int(blockIdx.x), kappa, S, ok, sm);
}

// The sum over the nodes for one particle (wrapped position xw, concentration
// kk) by S adjacent lanes, lane j summing the nodes k = j, j + S, j + 2S, ...
// in order (interleaved, so the S lanes read neighbouring LDS words instead
// of one bank); the S partial sums are combined by an xor butterfly, a fixed
// pairwise tree whose result every lane of the group holds. In the float form
// the loop runs over k = g - g0, so the table read is a broadcast and the
// field read is per lane. `tab`, `tf` and `etab` are the LDS tables of the
// nodes, the field and the exponential.
template <typename T>
__device__ __forceinline__ T gather_nodes(double xw, double kk, int j, int S, int M, double L, const SinCos<T>* tab,
                                          const T* tf, const double* etab) {
  PGeo<T> gp;
  make_geo(xw, L, M, gp);
  const T A = T(-2.0 * kk * Flt<T>::unit);
  const double w = (L / M) / (L * i0e_f64(kk));
  Acc<T> acc;
  acc.zero();
  if constexpr (std::is_same<T, float>::value) {
    // node g = g0 + k (mod M); groups of four without a bound test inside
    // a group keep their LDS reads in flight together (the run folds fall
    // after every kRun terms either way)
    auto term = [&](int k) {
      const SinCos<T> e = tab[k];
      const T s = e.s * gp.cb - e.c * gp.sb;
      const int g = gp.g0 + k;
      return tf[g >= M ? g - M : g] * Flt<T>::ex(A * (s * s), etab);
    };
    int k = j, q = 0;
    for (; k + 3 * S < M; k += 4 * S, q += 4) {
      T e[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) e[u] = term(k + u * S);
#pragma unroll
      for (int u = 0; u < 4; ++u) acc.add(e[u]);
      if (((q + 4) & (kRun - 1)) == 0) acc.fold();
    }
    for (; k < M; k += S, ++q) {
      acc.add(term(k));
      if ((q & (kRun - 1)) == kRun - 1) acc.fold();
    }
  } else if (__all(A >= T(-2.0 * kNearKappa))) {
    for (int g = j; g < M; g += S) {
      const T s = node_s(gp, g, M, tab);
      acc.add(tf[g] * Flt<T>::ex_in(A * (s * s), etab));
    }
  } else if (__all(A >= T(kExpTableMin))) {
    // sharp kernels in the wave: near nodes take the exact separation
    const double dx = L / double(M);
    const bool sharp = A < T(-2.0 * kNearKappa);
    for (int g = j; g < M; g += S) {
      T s = node_s(gp, g, M, tab);
      if (sharp) s = near_node_s(s, g, dx, gp.w, L);
      acc.add(tf[g] * Flt<T>::ex_in(A * (s * s), etab));
    }
  } else {
    const double dx = L / double(M);
    const bool sharp = A < T(-2.0 * kNearKappa);
    for (int g = j; g < M; g += S) {
      T s = node_s(gp, g, M, tab);
      if (sharp) s = near_node_s(s, g, dx, gp.w, L);
      acc.add(tf[g] * Flt<T>::ex(A * (s * s), etab));
    }
  }
  double tot = acc.value();
  for (int m = 1; m < S; m <<= 1) tot += __shfl_xor(tot, m, 64);
  return T(w * tot);
}

// The same for two particles of one thread (double): a node's reads serve both and
// their chains overlap. Every term and sum is gather_nodes'.
__device__ __forceinline__ void gather_nodes2(const double (&xw)[2], const double (&kk)[2], int M, double L,
                                              const SinCos<double>* tab, const double* tf, const double* etab,
                                              double (&out)[2]) {
  PGeo<double> gp[2];
  double A[2];
  Acc<double> acc[2];
  bool sharp[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    make_geo(xw[u], L, M, gp[u]);
    A[u] = -2.0 * kk[u] * Flt<double>::unit;
    sharp[u] = A[u] < -2.0 * kNearKappa;
    acc[u].zero();
  }
  const double dx = L / double(M);
  auto sum = [&](auto near, auto clamp) {
    for (int g = 0; g < M; ++g) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        double s = node_s(gp[u], g, M, tab);
        if (decltype(near)::value && sharp[u]) s = near_node_s(s, g, dx, gp[u].w, L);
        const double a = A[u] * (s * s);
        acc[u].add(tf[g] * (decltype(clamp)::value ? Flt<double>::ex(a, etab) : Flt<double>::ex_in(a, etab)));
      }
    }
  };
  if (__all(!sharp[0] && !sharp[1]))
    sum(std::false_type{}, std::false_type{});
  else if (__all(A[0] >= kExpTableMin && A[1] >= kExpTableMin))
    sum(std::true_type{}, std::false_type{});
  else
    sum(std::true_type{}, std::true_type{});
#pragma unroll
  for (int u = 0; u < 2; ++u) out[u] = (L / M) / (L * i0e_f64(kk[u])) * acc[u].value();
}

// S lanes per particle (1, 2, 4 or 8, from gather_split). Dynamic LDS: the
// node table (M SinCos<T>) and the field (M values of T).
template <typename T, int S>
__global__ void __launch_bounds__(kBlock) gather_kernel(const T* __restrict__ x, const T* __restrict__ kap,
                                                       double kappa_g, bool per, int64_t n, int M, double L,
                                                       const double* __restrict__ field, T* __restrict__ out,
                                                       uint32_t* status) {
  extern __shared__ __align__(16) unsigned char dyn[];
  __shared__ double etab[std::is_same<T, double>::value ? 256 : 1];
  SinCos<T>* tab = reinterpret_cast<SinCos<T>*>(dyn);
  T* tf = reinterpret_cast<T*>(tab + M);
  exp_table_fill<T>(etab);
  node_table(M, tab);
  for (int k = threadIdx.x; k < M; k += kBlock) tf[k] = T(field[k]);
  __syncthreads();
  const int64_t gid = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  const int64_t i = gid / S;
  if (i >= n) return;  // a particle's S lanes leave together
  const int j = int(gid % S);
  const double xi = double(x[i]);
  const double kk = per ? double(kap[i]) : kappa_g;
  if (j == 0) note_numeric(status, !isfinite(xi), per && !(isfinite(kk) && kk >= 0.0));
  const T v = gather_nodes<T>(xi - L * floor(xi / L), kk, j, S, M, L, tab, tf, etab);
  if (j == 0) out[i] = v;
}

// ------------------------------------- gather through the field's modes (double)
//
// With F^_m = (1/M) sum_g F_g exp(i 2 pi m g / M), which is periodic in m,
//   (L/M) sum_g F_g K_i(x_g - x_i) = F^_0 + 2 sum_{m>=1} rho_m(kappa_i) Re(F^_m exp(-i m theta_i)),
// an identity for every M and kappa_i (the aliases of the grid are the modes
// above M/2). Up to the order where rho_m falls below 1e-18 that is a third
// of the grid's nodes or less at ordinary widths, and a mode costs 9
// operations where a node costs 21: the backward recurrence t_{m-1} = t_{m+1}
// + (2m/kappa) t_m of t_m ~ I_m(kappa) (2), X <- X exp(-i theta) + t_m F^_m (6)
// and the largest part of X (1); out = (t_0 F^_0 + 2 Re X) / t_0. A workgroup
// makes the modes it needs itself (order x M multiply-adds, a few per cent
// of its work), so there is no scratch and no second launch.
//
// The rounding of the result is about half a unit of the series' size, |F^_0| and
// twice the largest part of X; that of the sum over the nodes is one or two units of
// G = sum |F_g| K_i. So a particle is taken whose value, or whose G (from the field's
// running sum of magnitudes over one and two of the kernel's widths), is at least
// 1/16 of the size; below (the empty stretch of a density), where the concentration
// needs too many modes and where anything is not finite it is listed and summed
// over the nodes as gather_kernel does. Against long double, 131,072 particles of
// kappa 14 to 68 on 256 nodes (over the nodes): four random modes and noise, error
// of the norm 2.6e-16 (3.1e-16), largest error 3.5e-15 G (2.3e-15); 1 + 0.95 cos 1.4e-16
// (2.8e-16) and 1.8e-15 (1.3e-15); a bump on a floor of 0.01 1.9e-16 (3.6e-16) and 3.2e-15
// (1.7e-15). Where the modes came from rotations and values of 1/256 were taken: 3.7e-16
// and 4.8e-15, 1.7e-16 and 4.8e-15, 2.4e-16 and 1.6e-14.
//
// The modes are scaled by a power of two (the field's largest node), so that neither
// a tiny field loses them nor a huge one overflows the recurrence.
// Bound by the FP64 vector pipe: 1,048,576 particles with concentrations of
// 14 to 68 on 256 nodes in 34 us (172 over the nodes), about half of it the 75
// modes, the rest the first reads (one round of workgroups, so nothing overlaps
// them), the tables, the modes' sums, the divisions and the listed particles.
constexpr int kGatherBlock = 512;    // threads
constexpr int kGatherModes = 1023;   // highest mode taken (kappa up to about 12,500)
constexpr double kGatherLow = 1.0 / 16.0;  // of the series' size
// Order from which rho_m(kappa) < 1e-18: m asinh(m/kappa) - sqrt(m^2 +
// kappa^2) + kappa, which bounds -log rho_m from below, is at least 41.45 at m
// = sqrt(83 (kappa + 7)) for every kappa (and the root of that bound is within
// 4 modes of it from kappa = 8 on); and the largest concentration an order serves.
__device__ __forceinline__ int gather_order(float kappa) { return int(ceilf(sqrtf(83.0f * (kappa + 7.0f)))) + 1; }
static double gather_kappa(int order) { return double(order - 2) * double(order - 2) / 83.0 - 7.0; }

// Dynamic LDS: the node table, the modes up to M/2 (double2), the field and the
// running sum of its magnitudes. P particles per thread.
template <int P>
__global__ void __launch_bounds__(kGatherBlock) gather_modes_kernel(const double* __restrict__ x,
                                                             const double* __restrict__ kap, double kappa_g, bool per,
                                                             int64_t n, int M, int cap, double kcap, double L,
                                                             const double* __restrict__ field,
                                                             double* __restrict__ out, uint32_t* status) {
  extern __shared__ __align__(16) unsigned char dyn[];
  __shared__ double2 unit[256];
  __shared__ double2 part[kGatherBlock];  // the modes' partial sums; then the list
  __shared__ double etab[256];
  static_assert(sizeof(part) >= 4 * kGatherBlock * sizeof(uint16_t));
  uint16_t* list = reinterpret_cast<uint16_t*>(part);
  __shared__ float kwave[kGatherBlock / 64], rwave[kGatherBlock / 64];
  __shared__ int ewave[kGatherBlock / 64], swave[kGatherBlock / 64];
  __shared__ int listed;
  SinCos<double>* tab = reinterpret_cast<SinCos<double>*>(dyn);
  double2* modes = reinterpret_cast<double2*>(tab + M);
  double* tf = reinterpret_cast<double*>(modes + M / 2 + 1);
  float* run = reinterpret_cast<float*>(tf + M);  // sum of |F_g|, g < k, scaled
  const int tid = threadIdx.x;
  const int64_t base = int64_t(blockIdx.x) * (P * kGatherBlock);
  const int cnt = int(min(int64_t(P * kGatherBlock), n - base));
  // the particles (in flight over the tables)
  double f1[P], kk[P];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int64_t i = base + min(p * kGatherBlock + tid, cnt - 1);
    f1[p] = x[i];
    kk[p] = per ? kap[i] : kappa_g;
  }
  if (tid == 0) listed = 0;
  unit_table_fill(unit);
  if (tid < kBlock) exp_table_fill<double>(etab);
  int fexp = -2000;
  for (int k = tid; k < M; k += kGatherBlock) {
    double sv, cv;
    sincospi(double(k) / double(M), &sv, &cv);
    tab[k] = SinCos<double>{sv, cv};
    const double v = field[k];
    tf[k] = v;
    if (v != 0.0) fexp = max(fexp, __builtin_amdgcn_frexp_exp(v));
  }
  // those the series does not serve keep kappa = -1
  float kmax = 0.0f;
  int served = 0;
  const double inv_L = 1.0 / L;
  const float node_width = float(M) * 0.15915494f;  // M / 2 pi: the kernel's width in nodes times sqrt(kappa)
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const bool finite = isfinite(f1[p]), serves = finite && kk[p] >= 0.0 && kk[p] <= kcap;
    note_numeric(status, !finite, per && !(isfinite(kk[p]) && kk[p] >= 0.0));
    f1[p] = period_fraction(f1[p], L, inv_L);
    if (serves) kmax = fmaxf(kmax, fmaxf(float(kk[p]), 1e-10f));
    served += __popcll(__ballot(serves));
    kk[p] = serves ? kk[p] : -1.0;
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    kmax = fmaxf(kmax, __shfl_xor(kmax, d, 64));
    fexp = max(fexp, __shfl_xor(fexp, d, 64));
  }
  if ((tid & 63) == 0) {
    kwave[tid >> 6] = kmax;
    ewave[tid >> 6] = fexp;
    swave[tid >> 6] = served;
  }
  __syncthreads();
  int all = 0;
#pragma unroll
  for (int w = 0; w < kGatherBlock / 64; ++w) {
    kmax = fmaxf(kmax, kwave[w]);
    fexp = max(fexp, ewave[w]);
    all += swave[w];
  }
  if (fexp == -2000) fexp = 0;  // (a field of zeros)
  {  // the running sum of |F|: a run of nodes per thread, the runs' sums by shuffles
    const int len = (M + kGatherBlock - 1) / kGatherBlock, lo = min(tid * len, M), hi = min(lo + len, M);
    float own = 0.0f;
    for (int k = lo; k < hi; ++k) own += fabsf(float(ldexp(tf[k], -fexp)));
    float sum = own;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const float o = __shfl_up(sum, d, 64);
      if ((tid & 63) >= d) sum += o;
    }
    if ((tid & 63) == 63) rwave[tid >> 6] = sum;
    __syncthreads();
    sum -= own;
    for (int w = 0; w < (tid >> 6); ++w) sum += rwave[w];
    for (int k = lo; k < hi; ++k) {
      run[k] = sum;
      sum += fabsf(float(ldexp(tf[k], -fexp)));
    }
    if (hi == M && lo < M) run[M] = sum;
    __syncthreads();
  }

  // the series runs for every particle, and the others are summed over the nodes
  // besides: taken where the nodes of those it serves (28 operations each) cost more
  const int ord = __builtin_amdgcn_readfirstlane(min(cap, gather_order(kmax)));
  if (kmax > 0.0f && 28.0f * float(M) * float(all) > 10.0f * float(ord) * float(P * kGatherBlock)) {  // (uniform)
    // F^_m, m = 0..min(ord, M/2) (the others are their conjugates): modes
    // side by side, the node pairs (g, M - g) in runs over the threads that
    // are left, every phase from the table (which holds half the circle), in four
    // sums each
    const int K = min(ord, M / 2) + 1, H = (M - 1) / 2;
    for (int m0 = 0; m0 < K; m0 += kGatherBlock) {
      const int kb = min(K - m0, kGatherBlock), S = kGatherBlock / kb;
      const int m = m0 + tid % kb, sub = tid / kb;
      double fr = 0.0, fi = 0.0;
      if (sub < S) {
        const int len = (H + S - 1) / S;
        const int lo = 1 + sub * len, hi = min(H, lo + len - 1);
        int idx = int((2u * unsigned(m) * unsigned(lo)) % unsigned(2 * M));
        double sr[4] = {0.0, 0.0, 0.0, 0.0}, si[4] = {0.0, 0.0, 0.0, 0.0};
        auto pair = [&](int g, int k) {
          const bool far = idx >= M;
          const SinCos<double> e = tab[far ? idx - M : idx];
          const double a = tf[g], b = tf[M - g];
          sr[k] = fma(far ? -e.c : e.c, a + b, sr[k]);
          si[k] = fma(far ? -e.s : e.s, a - b, si[k]);
          idx += 2 * m;
          idx -= idx >= 2 * M ? 2 * M : 0;
        };
        int g = lo;
        for (; g + 3 <= hi; g += 4) {
#pragma unroll
          for (int k = 0; k < 4; ++k) pair(g + k, k);
        }
        for (; g <= hi; ++g) pair(g, 0);
        fr = (sr[0] + sr[1]) + (sr[2] + sr[3]);
        fi = (si[0] + si[1]) + (si[2] + si[3]);
      }
      part[tid] = double2{fr, fi};
      __syncthreads();
      if (tid < kb) {
        fr = tf[0];
        fi = 0.0;
        double lr = 0.0, li = 0.0;
        if ((M & 1) == 0) add_exact(fr, (m & 1) ? -tf[M / 2] : tf[M / 2], lr);
        for (int q = 0; q < S; ++q) {
          add_exact(fr, part[q * kb + tid].x, lr);
          add_exact(fi, part[q * kb + tid].y, li);
        }
        fr = ldexp((fr + lr) / double(M), -fexp);
        fi = ldexp((fi + li) / double(M), -fexp);
        modes[m] = double2{fr, fi};
      }
      __syncthreads();
    }

    double c1[P], s1[P], ik[P], t[P], tp[P], xr[P], xi[P], mag[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const double2 z = table_phase(1.0, f1[p], unit);
      c1[p] = z.x;
      s1[p] = z.y;
      ik[p] = 1.0 / fmax(kk[p], 1e-18);  // (below, rho_1 = kappa / 2 is less than a rounding unit)
      t[p] = 1.0;
      tp[p] = xr[p] = xi[p] = mag[p] = 0.0;
    }
    // `parts` of X for its size: in turn, as it turns from mode to mode, and both
    // of the last eight
    auto mode = [&](int m, int j, double sign, int parts) {
      const double2 f = modes[j];
      const double fy = sign * f.y, m2 = double(2 * m);
#pragma unroll
      for (int p = 0; p < P; ++p) {
        const double r = fma(xr[p], c1[p], fma(xi[p], s1[p], t[p] * f.x));
        xi[p] = fma(xi[p], c1[p], fma(-xr[p], s1[p], t[p] * fy));
        xr[p] = r;
        if (parts & 1) mag[p] = fmax(mag[p], fabs(xr[p]));
        if (parts & 2) mag[p] = fmax(mag[p], fabs(xi[p]));
        const double tn = fma(m2 * ik[p], t[p], tp[p]);
        tp[p] = t[p];
        t[p] = tn;
      }
    };
    // t grows by at most 2 x 1023 x 1e18 a step: from 1e100 eight steps stay
    // finite, and one rescaling by 2^-600 brings the sum of them back
    auto rescale = [&]() {
      bool big = false;
#pragma unroll
      for (int p = 0; p < P; ++p) big = big || t[p] > 1e100;
      if (__any(big)) {
#pragma unroll
        for (int p = 0; p < P; ++p)
          if (t[p] > 1e100) {
            t[p] = ldexp(t[p], -600);
            tp[p] = ldexp(tp[p], -600);
            xr[p] = ldexp(xr[p], -600);
            xi[p] = ldexp(xi[p], -600);
            mag[p] = ldexp(mag[p], -600);
          }
      }
    };
    // runs of modes m whose remainder mod M rises to M/2 or falls to 0
    for (int m = ord; m > 8;) {  // (ord >= 26)
      const int r = m % M;
      const bool mirror = 2 * r > M;
      const int end = m - min(m - 8, mirror ? r - M / 2 : r + 1);
      int j = mirror ? M - r : r;
      const int step = mirror ? 1 : -1;
      const double sign = mirror ? -1.0 : 1.0;
      rescale();
      for (; (m - end) & 7; --m, j += step) mode(m, j, sign, 3);
      for (; m > end; m -= 8, j += 8 * step) {
        rescale();
#pragma unroll
        for (int u = 0; u < 8; ++u) mode(m - u, j + u * step, sign, 1 + (u & 1));
      }
    }
    rescale();
#pragma unroll 2
    for (int m = 8; m >= 1; --m) mode(m, m, 1.0, 3);
    const double f0 = modes[0].x;
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const int k = p * kGatherBlock + tid;
      const double v = fma(t[p], f0, 2.0 * fma(xr[p], c1[p], xi[p] * s1[p]));
      if (k < cnt) {
        const double whole = fma(t[p], fabs(f0), 2.0 * mag[p]);
        bool good = fabs(v) >= kGatherLow * whole;
        if (!good && whole > 0.0) {
          // of a width's peak, the nodes within one width have at least e^-1/2
          // and those within two at least e^-2
          const float u = float(f1[p]) * float(M), h = node_width * rsqrtf(fmaxf(float(kk[p]), 1.0f));
          auto within = [&](float reach) {
            const int a = int(ceilf(u - reach)), b = int(floorf(u + reach));
            float sum = run[min(max(b + 1, 0), M)] - run[min(max(a, 0), M)];
            if (a < 0) sum += run[M] - run[max(M + a, 0)];
            if (b >= M) sum += run[min(b + 1 - M, M)];
            return sum;
          };
          const float sum = 0.205f * within(h) + 0.136f * within(2.0f * h);
          good = double(sum) * t[p] >= kGatherLow * whole * double(h);
        }
        if (kk[p] >= 0.0 && good && whole < INFINITY && fabs(v) < INFINITY)
          out[base + k] = ldexp(v / t[p], fexp);
        else
          list[atomicAdd(&listed, 1)] = uint16_t(k);
      }
    }
  } else {
#pragma unroll
    for (int p = 0; p < P; ++p)
      if (p * kGatherBlock + tid < cnt) list[atomicAdd(&listed, 1)] = uint16_t(p * kGatherBlock + tid);
  }
  __syncthreads();
  // the listed ones over the nodes: their order in the list is not fixed,
  // their values do not depend on it
  const int nl = listed;
  if (nl == 0) return;
  int S = 1;
  while (S < 64 && 2 * S * (nl % (2 * kGatherBlock)) <= kGatherBlock) S *= 2;
  auto over_nodes = [&](int q, int lanes) {
    const int64_t i = base + list[q];
    const double xv = x[i];
    const int j = tid & (lanes - 1);
    const double v = gather_nodes<double>(xv - L * floor(xv / L), per ? kap[i] : kappa_g, j, lanes, M, L, tab, tf, etab);
    if (j == 0) out[i] = v;
  };
  int first = 0;  // of those not done two to a thread
  for (; first + 2 * kGatherBlock <= nl; first += 2 * kGatherBlock) {
    double xw[2], k2[2], v[2];
    int64_t i[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      i[u] = base + list[first + u * kGatherBlock + tid];
      const double xv = x[i[u]];
      xw[u] = xv - L * floor(xv / L);
      k2[u] = per ? kap[i[u]] : kappa_g;
    }
    gather_nodes2(xw, k2, M, L, tab, tf, etab, v);
#pragma unroll
    for (int u = 0; u < 2; ++u) out[i[u]] = v[u];
  }
  for (int q = first + tid / S; q < nl; q += kGatherBlock / S) over_nodes(q, S);
}

template <typename T>
__global__ void __launch_bounds__(kBlock) adapt_logsum_kernel(const T* __restrict__ x, int64_t n, int M, double L,
                                                             const double* __restrict__ pilot,
                                                             double* __restrict__ partials, uint32_t* status) {
  __shared__ double r0[kBlock / 64], r1[kBlock / 64];
  adapt_logsum_block<T>(x, n, M, L, pilot, blockIdx.x, partials + 2 * int64_t(blockIdx.x), r0, r1, status);
}

template <typename T>
__global__ void __launch_bounds__(kBlock) adapt_apply_kernel(const T* __restrict__ x, int64_t n, int M, double L,
                                                            const double* __restrict__ pilot, double kappa_star,
                                                            double alpha, const double* __restrict__ sums,
                                                            T* __restrict__ kout, double* __restrict__ log_g_out,
                                                            int64_t* __restrict__ nfl_out) {
  adapt_apply_block<T>(x, n, M, L, pilot, kappa_star, alpha, sums, blockIdx.x, kout);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (log_g_out) *log_g_out = sums[0] / double(n);
    if (nfl_out) *nfl_out = int64_t(sums[1]);
  }
}

// First-order (triangular) shape: the same chunked deposit with triangles
// (dev_tri.hpp), and a gather over the M nodes with the field in LDS.
template <typename T, bool PER, int G>
__global__ void __launch_bounds__(kBlock) tri_deposit_kernel(const T* __restrict__ x, const T* __restrict__ hi,
                                                            double h_g, int64_t n, int M, double L, int chunk,
                                                            double* __restrict__ partials, uint32_t* status) {
  __shared__ TriDepSmem<T> sm;
  const int64_t lo = int64_t(blockIdx.x) * chunk;
  const int cnt = int(min(int64_t(chunk), n - lo));
  tri_deposit_block<T, PER, G>(x, hi, h_g, M, L, lo, cnt, partials + int64_t(blockIdx.x) * M, sm, status);
}

template <typename T>
__global__ void __launch_bounds__(kBlock) tri_gather_kernel(const T* __restrict__ x, const T* __restrict__ hi,
                                                           double h_g, bool per, int64_t n, int M, double L,
                                                           const double* __restrict__ field, T* __restrict__ out,
                                                           uint32_t* status) {
  extern __shared__ __align__(16) unsigned char dyn[];
  T* tf = reinterpret_cast<T*>(dyn);
  for (int k = threadIdx.x; k < M; k += kBlock) tf[k] = T(field[k]);
  __syncthreads();
  const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (i >= n) return;
  const double h = per ? double(hi[i]) : h_g;
  note_numeric(status, !isfinite(double(x[i])), per && !(h > 0.0 && h <= 0.5 * L));
  const TriGeo<T> p = tri_geo<T>(double(x[i]), h, L, M);
  // a Kahan step per node: a support spans a few nodes, and runs with their
  // fold test were 15 % slower here in float
  SumOf<T> acc;
  auto add = [&](T v) { acc.add(v); };
  // Nodes beyond h / dx cells of the particle add exact zeros, so a
  // particle whose support is shorter than the circle visits only the nodes
  // g0 - r .. g0 + r (one node of margin against the rounding of q), still
  // in ascending node order: for a finite field the sum is the full
  // loop's, bit for bit.
  const int r = int(fmin(ceil(h * (double(M) / L)), double(M))) + 1;
  if (isfinite(double(p.w)) && 2 * r < M) {
    const int a = p.g0 - r, b = p.g0 + r;
    const int lo1 = a < 0 ? 0 : (b >= M ? 0 : a);
    const int hi1 = a < 0 ? b : (b >= M ? b - M : b);
    const int lo2 = a < 0 ? a + M : (b >= M ? a : M);
    for (int g = lo1; g <= hi1; ++g) add(tf[g] * tri_node(p, g, M));
    for (int g = lo2; g < M; ++g) add(tf[g] * tri_node(p, g, M));
  } else {
    for (int g = 0; g < M; ++g) add(tf[g] * tri_node(p, g, M));
  }
  out[i] = T((L / M) * double(p.w) * acc.value());
}

// ------------------------------------------------------------------ host

size_t deposit_workspace_bytes(int64_t n, int M) {
  const int64_t chunks = ceil_div(n, deposit_chunk(n));
  Carver c(nullptr, 0);
  c.take<double>(size_t(chunks) * M);
  c.take<double>(column_sum_scratch(chunks, M) / sizeof(double) + 1);
  return c.used;
}

size_t adapt_workspace_bytes(int64_t n) {
  const int64_t blocks = ceil_div(n, kBlock);
  Carver c(nullptr, 0);
  c.take<double>(size_t(blocks) * 2);
  c.take<double>(column_sum_scratch(blocks, 2) / sizeof(double) + 1);
  c.take<double>(2);
  return c.used;
}

template <typename T, bool PER>
static kde_status launch_deposit_t(const kde_domain* dom, int64_t n, const T* x, const T* kap, double kappa,
                                   double* partials, int chunk, int64_t chunks, hipStream_t s, uint32_t* status,
                                   TimedLaunch& timed, hipEvent_t start, const unsigned int* skip) {
  const int M = dom->M;
  const dim3 grid{unsigned(chunks)}, block{unsigned(kBlock)};
  const double kg = kappa;
  const size_t lds = dep_table_bytes<T>(n, M);
  KDE_RETURN_IF(check_lds(lds + sizeof(DepSmem<T>)));
  if (M <= kBlock) {
    hipExtLaunchKernelGGL((deposit_kernel<T, PER, 1>), grid, block, lds, s, start, timed.stop(), 0, x, kap, kg, n, M, dom->L, chunk, partials, status, skip);
  } else if (M <= 2 * kBlock) {
    hipExtLaunchKernelGGL((deposit_kernel<T, PER, 2>), grid, block, lds, s, start, timed.stop(), 0, x, kap, kg, n, M, dom->L, chunk, partials, status, skip);
  } else if (M <= 4 * kBlock) {
    hipExtLaunchKernelGGL((deposit_kernel<T, PER, 4>), grid, block, lds, s, start, timed.stop(), 0, x, kap, kg, n, M, dom->L, chunk, partials, status, skip);
  } else if (M <= 8 * kBlock) {
    hipExtLaunchKernelGGL((deposit_kernel<T, PER, 8>), grid, block, lds, s, start, timed.stop(), 0, x, kap, kg, n, M, dom->L, chunk, partials, status, skip);
  } else {
    hipExtLaunchKernelGGL((deposit_kernel<T, PER, 16>), grid, block, lds, s, start, timed.stop(), 0, x, kap, kg, n, M, dom->L, chunk, partials, status, skip);
  }
  KDE_CHECK_LAUNCH();
  return KDE_OK;
}

template <typename T, bool PER>
static kde_status launch_tri_deposit_t(const kde_domain* dom, int64_t n, const T* x, const T* hi, double h,
                                       double* partials, int chunk, int64_t chunks, hipStream_t s,
                                       uint32_t* status) {
  const int M = dom->M;
  const dim3 grid{unsigned(chunks)}, block{unsigned(kBlock)};
  KDE_RETURN_IF(check_lds(sizeof(TriDepSmem<T>)));
  TimedLaunch timed(KDE_KERNEL_DEPOSIT, s);
  if (M <= kBlock) {
    hipExtLaunchKernelGGL((tri_deposit_kernel<T, PER, 1>), grid, block, 0, s, timed.start(), timed.stop(), 0, x, hi, h, n, M, dom->L, chunk, partials, status);
  } else if (M <= 2 * kBlock) {
    hipExtLaunchKernelGGL((tri_deposit_kernel<T, PER, 2>), grid, block, 0, s, timed.start(), timed.stop(), 0, x, hi, h, n, M, dom->L, chunk, partials, status);
  } else if (M <= 4 * kBlock) {
    hipExtLaunchKernelGGL((tri_deposit_kernel<T, PER, 4>), grid, block, 0, s, timed.start(), timed.stop(), 0, x, hi, h, n, M, dom->L, chunk, partials, status);
  } else if (M <= 8 * kBlock) {
    hipExtLaunchKernelGGL((tri_deposit_kernel<T, PER, 8>), grid, block, 0, s, timed.start(), timed.stop(), 0, x, hi, h, n, M, dom->L, chunk, partials, status);
  } else {
    hipExtLaunchKernelGGL((tri_deposit_kernel<T, PER, 16>), grid, block, 0, s, timed.start(), timed.stop(), 0, x, hi, h, n, M, dom->L, chunk, partials, status);
  }
  KDE_CHECK_LAUNCH();
  return KDE_OK;
}

kde_status deposit(const kde_domain* dom, int64_t n, const void* x, const void* kap, double kappa, double* rho,
                   void* ws, size_t ws_bytes, hipStream_t s, uint32_t* status) {
  const int chunk = deposit_chunk(n);
  const int64_t chunks = ceil_div(n, chunk);
  Carver c(ws, ws_bytes);
  double* partials = c.take<double>(size_t(chunks) * dom->M);
  const size_t sums = column_sum_scratch(chunks, dom->M) / sizeof(double);
  double* scratch = c.take<double>(sums + 1);
  if (!c.fits()) return fail(KDE_E_WORKSPACE, "workspace too small: %zu < %zu bytes", ws_bytes, c.used);
  const unsigned int* skip = nullptr;
  if (dom->shape == KDE_SHAPE_TRIANGLE) {
    if (dom->prec == KDE_F64) {
      const double* xx = static_cast<const double*>(x);
      const double* hh = static_cast<const double*>(kap);
      KDE_RETURN_IF((hh ? launch_tri_deposit_t<double, true>(dom, n, xx, hh, kappa, partials, chunk, chunks, s, status)
                        : launch_tri_deposit_t<double, false>(dom, n, xx, hh, kappa, partials, chunk, chunks, s, status)));
    } else {
      const float* xx = static_cast<const float*>(x);
      const float* hh = static_cast<const float*>(kap);
      KDE_RETURN_IF((hh ? launch_tri_deposit_t<float, true>(dom, n, xx, hh, kappa, partials, chunk, chunks, s, status)
                        : launch_tri_deposit_t<float, false>(dom, n, xx, hh, kappa, partials, chunk, chunks, s, status)));
    }
  } else {
    TimedLaunch timed(KDE_KERNEL_DEPOSIT, s);
    hipEvent_t start = timed.start();
    const int order = kap ? 0 : fourier_order(kappa);
    if (!kap && deposit_tries_moments(dom->prec, n, dom->M) && order <= kNarrowMax) {
      // their partial rows (at most 256 of 2 kNarrowMax), sums and series fit the rows
      // of the sum over the particles (n M >= 2^25: at least 2^16 doubles),
      // which overwrites them if it has to run; the word behind the column
      // sums' scratch is nobody else's
      static_assert(size_t(kMomChunks) * 2 * kNarrowMax + kNarrowSums <= (size_t(1) << 25) / kDepMaxChunk);
      double* S = partials + size_t(kMomChunks) * 2 * kNarrowMax;
      unsigned int* ok = reinterpret_cast<unsigned int*>(scratch + sums);
      const ScanBufs mom{narrow_plan(n, order), partials, S, ok};
      KDE_RETURN_IF(check_lds(sizeof(double2) * size_t(dom->M) + sizeof(SynthSmem)));
      KDE_RETURN_IF(launch_moment_rows(static_cast<const double*>(x), n, dom->L, mom, s, start, nullptr, status));
      hipLaunchKernelGGL(deposit_sums_kernel, dim3(unsigned(narrow_units(order))), dim3(kBlock), 0, s,
                         (const double*)partials, mom.plan.rows, order, kappa, S, ok);
      KDE_CHECK_LAUNCH();
      hipLaunchKernelGGL(deposit_synthesis_kernel, dim3(unsigned(synthesis_parts(dom->M))), dim3(kBlock),
                         sizeof(double2) * size_t(dom->M), s, (const double*)S, order, double(n), dom->L, dom->M, rho, ok);
      KDE_CHECK_LAUNCH();
      start = nullptr;
      skip = ok;
    }
    if (dom->prec == KDE_F64) {
      const double* xx = static_cast<const double*>(x);
      const double* kk = static_cast<const double*>(kap);
      KDE_RETURN_IF((kk ? launch_deposit_t<double, true>(dom, n, xx, kk, kappa, partials, chunk, chunks, s, status, timed, start, skip)
                        : launch_deposit_t<double, false>(dom, n, xx, kk, kappa, partials, chunk, chunks, s, status, timed, start, skip)));
    } else {
      const float* xx = static_cast<const float*>(x);
      const float* kk = static_cast<const float*>(kap);
      KDE_RETURN_IF((kk ? launch_deposit_t<float, true>(dom, n, xx, kk, kappa, partials, chunk, chunks, s, status, timed, start, skip)
                        : launch_deposit_t<float, false>(dom, n, xx, kk, kappa, partials, chunk, chunks, s, status, timed, start, skip)));
    }
  }
  return launch_column_sum(partials, chunks, dom->M, scratch, rho, s, 1.0 / double(n), skip);
}

// Lanes per particle for the gather: split the node loop while the
// particles alone would leave the chip short of workgroups (fewer than
// 1024) and every lane keeps at least 32 nodes.
static int gather_split(int64_t n, int M) {
  int S = 1;
  while (S < 8 && M / (2 * S) >= 32 && ceil_div(n * S, kBlock) < 1024) S *= 2;
  return S;
}

// The double gather goes through the modes from 2^25 (particle, node) pairs
// on, on grids with at least 8 particles per node (each workgroup makes its
// modes), of at least 64 nodes with one concentration and 256 with per-
// particle ones, which only the device sees. 131,072 particles on 256 nodes:
// 11.2 us at kappa = 26 (29 over the nodes), 22.6 at 300 (34), 29.6 at 700 (34),
// 34.8 at 1200 (34); 16,000 on 256: 11.3 (8.0); 40,000 on 4096: 109 at 300 (350). The
// series is taken up to 7/4 M modes, where it costs what the nodes do; a workgroup
// whose particles are mostly sharper sums all of them over the nodes, two to a
// thread: 1,048,576 on 256 nodes all above 1500 (a kernel about as narrow as the
// spacing) 218 us (190), 131,072 all above 10,000 43 us (34). 4, 2 or 1
// particles per thread by what fills the chip with two workgroups per CU.
constexpr int kGatherFrom = 64, kGatherPerFrom = 256;
constexpr int64_t kGatherPairs = int64_t(1) << 25;
constexpr int64_t kGatherSpread = 512 * kGatherBlock;

template <typename T>
static kde_status launch_gather_t(const kde_domain* dom, int64_t n, const T* x, const T* kap, double kappa,
                                  const double* field, T* out, size_t lds, hipStream_t s, uint32_t* status) {
  const dim3 block{unsigned(kBlock)};
  const bool per = kap != nullptr;
  if constexpr (std::is_same<T, double>::value) {
    const int cap = std::min(dom->M + dom->M / 4 * 3, kGatherModes);
    const double kcap = gather_kappa(cap);
    if (dom->M >= (per ? kGatherPerFrom : kGatherFrom) && n >= 8 * int64_t(dom->M) &&
        n * dom->M >= kGatherPairs && (per || kappa <= kcap)) {
      const size_t tables = size_t(dom->M) * 3 * sizeof(double) + size_t(dom->M / 2 + 1) * sizeof(double2);
      const size_t fixed = 256 * (sizeof(double2) + sizeof(double)) + kGatherBlock * sizeof(double2) + 128;
      const size_t runs = (size_t(dom->M) + 1) * sizeof(float);
      const size_t modes = tables + runs;
      KDE_RETURN_IF(check_lds(modes + fixed));
      TimedLaunch timed(KDE_KERNEL_GATHER, s);
      if (2 * n > 3 * kGatherSpread)
        hipExtLaunchKernelGGL(gather_modes_kernel<4>, dim3(unsigned(ceil_div(n, 4 * kGatherBlock))), dim3(kGatherBlock), modes, s, timed.start(), timed.stop(), 0, x, kap, kappa, per, n, dom->M, cap, kcap, dom->L, field, out, status);
      else if (n > kGatherSpread)
        hipExtLaunchKernelGGL(gather_modes_kernel<2>, dim3(unsigned(ceil_div(n, 2 * kGatherBlock))), dim3(kGatherBlock), modes, s, timed.start(), timed.stop(), 0, x, kap, kappa, per, n, dom->M, cap, kcap, dom->L, field, out, status);
      else
        hipExtLaunchKernelGGL(gather_modes_kernel<1>, dim3(unsigned(ceil_div(n, kGatherBlock))), dim3(kGatherBlock), modes, s, timed.start(), timed.stop(), 0, x, kap, kappa, per, n, dom->M, cap, kcap, dom->L, field, out, status);
      KDE_CHECK_LAUNCH();
      return KDE_OK;
    }
  }
  const int S = gather_split(n, dom->M);
  const dim3 grid{unsigned(ceil_div(n * S, kBlock))};
  TimedLaunch timed(KDE_KERNEL_GATHER, s);
  switch (S) {
    case 1:
      hipExtLaunchKernelGGL((gather_kernel<T, 1>), grid, block, lds, s, timed.start(), timed.stop(), 0, x, kap, kappa, per, n, dom->M, dom->L, field, out, status);
      break;
    case 2:
      hipExtLaunchKernelGGL((gather_kernel<T, 2>), grid, block, lds, s, timed.start(), timed.stop(), 0, x, kap, kappa, per, n, dom->M, dom->L, field, out, status);
      break;
    case 4:
      hipExtLaunchKernelGGL((gather_kernel<T, 4>), grid, block, lds, s, timed.start(), timed.stop(), 0, x, kap, kappa, per, n, dom->M, dom->L, field, out, status);
      break;
    default:
      hipExtLaunchKernelGGL((gather_kernel<T, 8>), grid, block, lds, s, timed.start(), timed.stop(), 0, x, kap, kappa, per, n, dom->M, dom->L, field, out, status);
      break;
  }
  KDE_CHECK_LAUNCH();
  return KDE_OK;
}

kde_status gather(const kde_domain* dom, int64_t n, const void* x, const void* kap, double kappa,
                  const double* field, void* out, hipStream_t s, uint32_t* status) {
  const dim3 grid{unsigned(ceil_div(n, kBlock))}, block{unsigned(kBlock)};
  if (dom->shape == KDE_SHAPE_TRIANGLE) {
    const size_t lds = size_t(dom->M) * elem_size(dom->prec);
    KDE_RETURN_IF(check_lds(lds));
    TimedLaunch timed(KDE_KERNEL_GATHER, s);
    if (dom->prec == KDE_F64)
      hipExtLaunchKernelGGL(tri_gather_kernel<double>, grid, block, lds, s, timed.start(), timed.stop(), 0,
                         static_cast<const double*>(x),
                         static_cast<const double*>(kap), kappa, kap != nullptr, n, dom->M, dom->L, field,
                         static_cast<double*>(out), status);
    else
      hipExtLaunchKernelGGL(tri_gather_kernel<float>, grid, block, lds, s, timed.start(), timed.stop(), 0,
                         static_cast<const float*>(x),
                         static_cast<const float*>(kap), kappa, kap != nullptr, n, dom->M, dom->L, field,
                         static_cast<float*>(out), status);
    KDE_CHECK_LAUNCH();
    return KDE_OK;
  }
  const size_t lds = 3 * size_t(dom->M) * elem_size(dom->prec);
  KDE_RETURN_IF(check_lds(lds + (dom->prec == KDE_F64 ? 256 * sizeof(double) : sizeof(double))));  // + exp table
  if (dom->prec == KDE_F64)
    KDE_RETURN_IF(launch_gather_t<double>(dom, n, static_cast<const double*>(x), static_cast<const double*>(kap),
                                          kappa, field, static_cast<double*>(out), lds, s, status));
  else
    KDE_RETURN_IF(launch_gather_t<float>(dom, n, static_cast<const float*>(x), static_cast<const float*>(kap),
                                         kappa, field, static_cast<float*>(out), lds, s, status));
  return KDE_OK;
}

kde_status adapt_widths(const kde_domain* dom, int64_t n, const void* x, const double* pilot, double kappa_star,
                        double alpha, void* kout, double* log_g, int64_t* nfl, void* ws, size_t ws_bytes,
                        hipStream_t s, uint32_t* status) {
  const int64_t blocks = ceil_div(n, kBlock);
  Carver c(ws, ws_bytes);
  double* partials = c.take<double>(size_t(blocks) * 2);
  double* scratch = c.take<double>(column_sum_scratch(blocks, 2) / sizeof(double) + 1);
  double* sums = c.take<double>(2);
  if (!c.fits()) return fail(KDE_E_WORKSPACE, "workspace too small: %zu < %zu bytes", ws_bytes, c.used);
  const dim3 grid{unsigned(blocks)}, block{unsigned(kBlock)};
  TimedLaunch timed(KDE_KERNEL_ADAPT, s);  // from the log sums' start to the widths' end
  if (dom->prec == KDE_F64) {
    hipExtLaunchKernelGGL(adapt_logsum_kernel<double>, grid, block, 0, s, timed.start(), nullptr, 0,
                          static_cast<const double*>(x), n, dom->M, dom->L, pilot, partials, status);
  } else {
    hipExtLaunchKernelGGL(adapt_logsum_kernel<float>, grid, block, 0, s, timed.start(), nullptr, 0,
                          static_cast<const float*>(x), n, dom->M, dom->L, pilot, partials, status);
  }
  KDE_CHECK_LAUNCH();
  KDE_RETURN_IF(launch_column_sum(partials, blocks, 2, scratch, sums, s));
  if (dom->prec == KDE_F64) {
    hipExtLaunchKernelGGL(adapt_apply_kernel<double>, grid, block, 0, s, nullptr, timed.stop(), 0,
                          static_cast<const double*>(x), n, dom->M, dom->L, pilot, kappa_star, alpha,
                          (const double*)sums, static_cast<double*>(kout), log_g, nfl);
  } else {
    hipExtLaunchKernelGGL(adapt_apply_kernel<float>, grid, block, 0, s, nullptr, timed.stop(), 0,
                          static_cast<const float*>(x), n, dom->M, dom->L, pilot, kappa_star, alpha,
                          (const double*)sums, static_cast<float*>(kout), log_g, nfl);
  }
  KDE_CHECK_LAUNCH();
  return KDE_OK;
}

}  // namespace kde
