// One-set launchers of the particle layout (wrap, pack, stable counting sort
// by angular cell; the device pieces are in dev_layout.hpp) and of the
// fixed-order column sums (dev_reduce.hpp).
//
// The pair sums of the CV objective do not depend on particle order, but a
// wavefront of neighbouring particles lets the pair kernel stop early for
// concentrations at which every pair of the wave is negligible. The sort is
// stable and uses only integer atomics for the histogram counts, so the
// resulting order (and every rounding downstream) is deterministic.
#include "dev_layout.hpp"
#include "dev_reduce.hpp"

namespace kde {

SortPlan make_sort_plan(int64_t n) {
  SortPlan p;
  p.n = n;
  int64_t cells = n / 32;
  if (cells < 1) cells = 1;
  if (cells > 8192) cells = 8192;
  p.cells = int(cells);
  int64_t blocks = ceil_div(n, 2048);
  if (blocks < 1) blocks = 1;
  if (blocks > 128) blocks = 128;
  p.blocks = int(blocks);
  p.chunk = ceil_div(n, blocks);
  return p;
}



// Per-block histogram over its contiguous chunk; hist is cell-major
// [cells][blocks] so that one exclusive scan yields stable scatter bases.
template <typename T>
__global__ void __launch_bounds__(kBlock) sort_hist_kernel(const T* __restrict__ x, int64_t n, double L,
                                                          int cells, int64_t chunk,
                                                          int32_t* __restrict__ hist, uint32_t* status) {
  extern __shared__ int32_t lh[];
  const int64_t lo = int64_t(blockIdx.x) * chunk;
  sort_hist_block<T>(x, lo, min(n, lo + chunk), L, cells, blockIdx.x, gridDim.x, lh, hist, status);
}

__global__ void __launch_bounds__(kBlock) exclusive_scan_kernel(int32_t* __restrict__ a, int64_t len) {
  __shared__ int tot[kBlock / 64];
  block_scan_global(a, len, tot);
}

// Stable scatter: the block walks its chunk in rounds of 256 particles; a
// particle's rank among equal cells comes from the lanes before it in its
// wave plus the counts already placed by earlier waves and rounds.
template <typename T, typename P>
__global__ void __launch_bounds__(kBlock) sort_scatter_kernel(const T* __restrict__ x, int64_t n, double L,
                                                             int cells, int64_t chunk,
                                                             const int32_t* __restrict__ base_in,
                                                             P* __restrict__ packed,
                                                             int32_t* __restrict__ perm) {
  extern __shared__ int32_t base[];
  const int64_t lo = int64_t(blockIdx.x) * chunk;
  sort_scatter_block<T, P>(x, lo, min(n, lo + chunk), L, cells, blockIdx.x, gridDim.x, base_in, base, packed, perm);
}

template <typename T, typename P>
kde_status launch_pack_sorted_as(const T* x, int64_t n, double L, const SortPlan& plan, int32_t* hist, P* packed,
                                 int32_t* perm, hipStream_t s, uint32_t* status) {
  const size_t lds = size_t(plan.cells) * sizeof(int32_t);
  hipLaunchKernelGGL(sort_hist_kernel<T>, dim3(plan.blocks), dim3(kBlock), lds, s, x, n, L,
                     plan.cells, plan.chunk, hist, status);
  KDE_CHECK_LAUNCH();
  hipLaunchKernelGGL(exclusive_scan_kernel, dim3(1), dim3(kBlock), 0, s, hist,
                     int64_t(plan.cells) * plan.blocks);
  KDE_CHECK_LAUNCH();
  hipLaunchKernelGGL((sort_scatter_kernel<T, P>), dim3(plan.blocks), dim3(kBlock), lds, s, x, n, L,
                     plan.cells, plan.chunk, hist, packed, perm);
  KDE_CHECK_LAUNCH();
  return KDE_OK;
}

template kde_status launch_pack_sorted_as<double, double>(const double*, int64_t, double, const SortPlan&, int32_t*,
                                                          double*, int32_t*, hipStream_t, uint32_t*);
template kde_status launch_pack_sorted_as<float, uint32_t>(const float*, int64_t, double, const SortPlan&, int32_t*,
                                                           uint32_t*, int32_t*, hipStream_t, uint32_t*);

// ------------------------------------------------------ deterministic sums

// Block (row block x, column block y): one column per thread, kSumCols
// columns per workgroup, so a wide sum spreads its reads over
// ceil(cols / kSumCols) workgroups per row block.
constexpr int kSumCols = 64;

__global__ void __launch_bounds__(kSumCols) colsum_level1_kernel(const double* __restrict__ in, int64_t rows,
                                                                int cols, double* __restrict__ l1,
                                                                const unsigned int* skip) {
  if (skip && *skip) return;
  const int c = int(blockIdx.y) * kSumCols + threadIdx.x;
  if (c < cols) l1[int64_t(blockIdx.x) * cols + c] = colsum_level1(in, rows, cols, blockIdx.x, c);
}

__global__ void __launch_bounds__(kSumCols) colsum_level2_kernel(const double* __restrict__ l1, int64_t g, int cols,
                                                                double scale, double* __restrict__ out,
                                                                const unsigned int* skip) {
  if (skip && *skip) return;
  const int c = int(blockIdx.x) * kSumCols + threadIdx.x;
  if (c < cols) out[c] = colsum_level2(l1, g, cols, c, scale);
}

// Both levels at once when there is one row block (and more columns than the
// fused kernel takes): level 2 over a single
// level-1 row is 0 + l1, exactly l1, so out[c] = l1 * scale has the
// two-kernel result's bits.
__global__ void __launch_bounds__(kSumCols) colsum_single_kernel(const double* __restrict__ in, int64_t rows,
                                                                int cols, double scale, double* __restrict__ out,
                                                                const unsigned int* skip) {
  if (skip && *skip) return;
  const int c = int(blockIdx.x) * kSumCols + threadIdx.x;
  if (c < cols) out[c] = colsum_level1(in, rows, cols, 0, c) * scale;
}

// Both levels by one workgroup per column: its threads fetch the column into
// LDS, thread b adds row block b, and the row blocks' sums are added up: level
// 1's and level 2's additions in their order, so the two kernels' bits,
// without a second launch and without waiting for memory every kLoadAhead
// rows. The 16 columns of a cache line run on one XCD (workgroups go to the
// XCDs in turn), whose L2 fetches the line once. 2033 rows of 128 columns, a float
// deposit's: 5.6 us against 4.3 + 3.9 and the gap between them (two, four and
// eight columns per workgroup: 6.2, 7.5 and 8.2); 4096 rows of two, the widths':
// 4.4 against 4.1 + 2. With 8192 rows (4,194,304 particles) of 64 columns the
// deposit is 8 % slower with it (too few CUs read), with 1024 columns and more
// (a lane's reads no longer share lines in time) 3 to 7 %; up to 4096 rows of 512
// columns it is 0 to 60 % faster (20,000 on 64 nodes 13.4 -> 8.3 us, 1,048,576
// on 256 82.7 -> 72.7). Few rows gain too: the 28 of a 1780-particle float scan
// took 8.6 us, each waiting for memory in turn, now 4.5 (8000 on 64 nodes 13.7 -> 8.2).
constexpr int kFuseThreads = 512;
constexpr int64_t kFuseRows = 4096;
constexpr int kFuseCols = 512;
constexpr int kLineCols = 16, kXcds = 8;

__device__ __forceinline__ int fuse_slot(int r) { return r + r / kSumRows; }  // a word of padding per row block

__global__ void __launch_bounds__(kFuseThreads) colsum_fused_kernel(const double* __restrict__ in, int rows, int cols,
                                                                   double scale, double* __restrict__ out,
                                                                   const unsigned int* skip) {
  __shared__ double column[kFuseRows + kFuseRows / kSumRows];
  __shared__ double l1[kFuseRows / kSumRows];
  if (skip && *skip) return;
  const int turn = int(blockIdx.x) / kXcds;
  const int c = (turn / kLineCols * kXcds + int(blockIdx.x) % kXcds) * kLineCols + turn % kLineCols;
  if (c >= cols) return;
  const int g = (rows + kSumRows - 1) / kSumRows;
#pragma unroll 8
  for (int r = threadIdx.x; r < rows; r += kFuseThreads) column[fuse_slot(r)] = in[int64_t(r) * cols + c];
  __syncthreads();
  if (int(threadIdx.x) < g) {
    const int r0 = int(threadIdx.x) * kSumRows, n = min(rows - r0, kSumRows);
    const double* p = column + fuse_slot(r0);
    double s = 0.0;
#pragma unroll 16
    for (int r = 0; r < n; ++r) s += p[r];
    l1[threadIdx.x] = s;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int k = 0; k < g; ++k) s += l1[k];
    out[c] = s * scale;
  }
}

size_t column_sum_scratch(int64_t rows, int cols) {
  return size_t(ceil_div(rows, kSumRows)) * size_t(cols) * sizeof(double);
}

kde_status launch_column_sum(const double* in, int64_t rows, int cols, double* scratch, double* out, hipStream_t s,
                             double scale, const unsigned int* skip) {
  const int64_t g = ceil_div(rows, kSumRows);
  const unsigned cb = unsigned(ceil_div(cols, kSumCols));
  if (rows <= kFuseRows && cols <= kFuseCols) {
    const unsigned lines = unsigned(ceil_div(ceil_div(cols, kLineCols), kXcds) * kXcds);
    hipLaunchKernelGGL(colsum_fused_kernel, dim3(lines * kLineCols), dim3(kFuseThreads), 0, s, in, int(rows), cols,
                       scale, out, skip);
    KDE_CHECK_LAUNCH();
    return KDE_OK;
  }
  if (g == 1) {
    hipLaunchKernelGGL(colsum_single_kernel, dim3(cb), dim3(kSumCols), 0, s, in, rows, cols, scale, out, skip);
    KDE_CHECK_LAUNCH();
    return KDE_OK;
  }
  hipLaunchKernelGGL(colsum_level1_kernel, dim3(unsigned(g), cb), dim3(kSumCols), 0, s, in, rows, cols, scratch, skip);
  KDE_CHECK_LAUNCH();
  hipLaunchKernelGGL(colsum_level2_kernel, dim3(cb), dim3(kSumCols), 0, s, (const double*)scratch, g, cols, scale,
                     out, skip);
  KDE_CHECK_LAUNCH();
  return KDE_OK;
}

}  // namespace kde
