// The host's rules of the Fourier-moment routes (csrc/dev_fourier.hpp).
#include <climits>
#include <cmath>
#include <cstdio>
#include <limits>

#include "dev_fourier.hpp"

using namespace kde;

static int failures = 0;
#define EXPECT(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); ++failures; } } while (0)

// The order of every concentration an entry point accepts: 1 for the
// smallest, growing with kappa, and beyond the longest series never short.
static void orders() {
  for (double k : {0.0, 5e-324, 1e-300, 1e-160, 1e-101, 1e-99, 1e-20}) EXPECT(fourier_order(k) == 1);
  int last = 1;
  for (double k = 1e-20; k <= KDE_MAX_FOURIER_KAPPA; k *= 1.01) {
    const int m = fourier_order(k);
    EXPECT(m >= last && m < 20000);
    last = m;
  }
  EXPECT(last > 9000);
  for (double k : {1.0001e6, 1e7, 1e12, 1e15, 5e16, 6e16, 1e17, 1e18, 1e33, 1e34, 1e100, 1e300,
                   std::numeric_limits<double>::max()})
    EXPECT(fourier_order(k) == INT_MAX);
  // where the narrow form ends
  EXPECT(fourier_order(144.5) == kNarrowMax && fourier_order(145.0) == kNarrowMax + 1);
}

// The refinement's arrays hold every series of a bracket, whose ends it
// evaluates at exp(log(kappa)): a few rounding units about kappa.
static void bracket_lengths() {
  int longer = 0;
  auto check = [&](double k) {
    double up = std::exp(std::log(k));
    for (int u = 0; u < 4; ++u) up = std::nextafter(up, INFINITY);
    for (int M : {fourier_order(k), fourier_order(k) - 1}) {  // (the refinement's may be one less)
      longer += series_length(M, up) > series_length(M, k);
      EXPECT(series_length(M, up) + 1 <= series_slots(M, k));  // its indices 0 .. length
    }
  };
  for (int k = 1; k <= 1000000; ++k) check(double(k));
  for (double k = 1e-3; k <= 1e6; k *= 1.00037) check(k);
  EXPECT(longer > 0);  // the case is met
}

// A plan covers the particles and the modes, and its arrays fit the room that
// they were planned for, down to the room for a single row.
static void plans() {
  for (int64_t n : {2, 63, 700, 4096, 12000, 20011, 65536, 1000003, 1 << 30}) {
    for (int M : {1, 4, 5, 111, 112, 113, 263, 264, 500, 759, 911, 1007, 1008, 4000, 9105}) {
      for (double rows : {1.0, 1.9, 2.0, 3.0, 7.5, 40.0, 300.0}) {
        const size_t room = 512 + size_t((rows + 1.0) * 16.0 * M);
        Carver c(nullptr, 0);
        const ScanBufs b = carve_scan(c, room, n, M);
        const MomentPlan& p = b.plan;
        EXPECT(c.used <= room && p.rows == p.chunks && p.M == M);
        EXPECT(p.chunks * p.per >= n && (p.chunks - 1) * p.per < n);
        if (p.direct) {
          EXPECT(p.mblocks * int64_t(p.direct) >= M && p.chunks == 1);
        } else if (p.narrow) {
          EXPECT(M <= kNarrowMax && kNarrowStep * (p.na - 1) + kNarrowB - 1 >= M && p.na <= kNarrowA);
        } else {
          const int values = 8 * p.tiles * p.mblocks;  // of a; modes kWideStep a +- b
          EXPECT(kWideStep * (values - 1) + kWideB - 1 >= M && p.tiles * p.ks <= 4 && 8 * p.tiles <= kWideA);
          EXPECT(p.per % (2 * kMomGroup) == 0);
        }
      }
    }
  }
}

// Which leading concentrations of a list go through the moments.
static void lists() {
  const double one[] = {0.3, 1.0, 3.7, 13.9, 51.8, 193.0, 720.0, 2683.0, 1e4};
  EXPECT(scan_fourier_count(KDE_F32, 65536, one, 9) == 0);
  EXPECT(scan_fourier_count(KDE_F64, 65536, one, 9) == 9);
  EXPECT(scan_fourier_count(KDE_F64, 64, one, 4) == 4);   // all below (64 / 3 pi)^2 = 46.1
  EXPECT(scan_fourier_count(KDE_F64, 64, one + 1, 8) == 0);  // three of eight: two passes of the rest as of all
  EXPECT(scan_fourier_count(KDE_F64, 64, one, 9) == 4);      // nine are three passes, the other five two
  EXPECT(scan_fourier_count(KDE_F64, 257, one + 1, 8) == 6 && scan_fourier_count(KDE_F64, 10, one, 9) == 0);
}

int main() {
  lists();
  plans();
  orders();
  bracket_lengths();
  if (failures == 0) std::printf("fourier rules ok\n");
  return failures ? 1 : 0;
}
