// Dense (plain-method) aggregation and disaggregation, eqs. (3) and (5), Figs. 2(a)
// and 3(a).  All kernels are pure HBM streams over the far-field array [N][2][N_dir] (a
// group's rows are contiguous):
//   aggregation    F[g][col] = sum_n A[n][col] x[n]
//   disaggregation V[n] = sum_col conj(A[n][col]) G[g][col]
// With one right-hand side they run on the vector units: the aggregation a column per
// lane, the disaggregation a row per wavefront.  With more, up to 8 right-hand sides share
// a read of A and the products run on the matrix cores (16 real columns hold the real and
// imaginary parts of 8 right-hand sides), which leaves the vector registers to loads in
// flight; the aggregation of groups of few rows stays on the vector units for up to 4.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "cplx.hpp"
#include "kernels.hpp"

namespace tuckfmm {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

// Aggregation with one right-hand side.  A workgroup takes 64 kCols columns of a group;
// its four wavefronts take the group's rows in turn and meet in LDS, so that a layout of
// few groups still fills the chip (24 groups of 909 rows and 5700 columns, complex128: 452 us
// with a thread per column and all rows in one wavefront, in 288 workgroups, about 310 now).
template <typename T>
__global__ __launch_bounds__(kThreads) void dense_agg_kernel(const typename Tr<T>::c* __restrict__ A,
                                                             const DenseGroup* __restrict__ groups, int n_chunks,
                                                             int ncols, const typename Tr<T>::c* __restrict__ x,
                                                             typename Tr<T>::c* __restrict__ F) {
  using C = typename Tr<T>::c;
  constexpr int kCols = 2 * Tr<T>::E;  // columns per lane
  constexpr int U = 4;                 // rows in flight
  __shared__ C sum[kWaves - 1][64 * kCols];
  const int g = blockIdx.x / n_chunks;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int c0 = (blockIdx.x - g * n_chunks) * 64 * kCols + lane;
  const DenseGroup grp = groups[g];
  C acc[kCols];
  int off[kCols];
#pragma unroll
  for (int j = 0; j < kCols; ++j) {
    acc[j] = czero<C>();
    off[j] = min(c0 + 64 * j, ncols - 1);  // (columns past the end are not stored)
  }
  const C* base = A + grp.row0 * ncols;
  const C* xb = x + grp.row0;
  int n = w;
  for (; n + kWaves * (U - 1) < grp.nb; n += kWaves * U) {
    C a[U][kCols];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int j = 0; j < kCols; ++j) a[u][j] = base[(int64_t)(n + kWaves * u) * ncols + off[j]];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const C xn = xb[n + kWaves * u];
#pragma unroll
      for (int j = 0; j < kCols; ++j) cfma(acc[j], a[u][j], xn);
    }
  }
  for (; n < grp.nb; n += kWaves) {
    const C xn = xb[n];
#pragma unroll
    for (int j = 0; j < kCols; ++j) cfma(acc[j], base[(int64_t)n * ncols + off[j]], xn);
  }
  if (w > 0) {
#pragma unroll
    for (int j = 0; j < kCols; ++j) sum[w - 1][64 * j + lane] = acc[j];
  }
  __syncthreads();
  if (w > 0) return;
#pragma unroll
  for (int j = 0; j < kCols; ++j) {
#pragma unroll
    for (int v = 0; v < kWaves - 1; ++v) {
      acc[j].x += sum[v][64 * j + lane].x;
      acc[j].y += sum[v][64 * j + lane].y;
    }
    if (c0 + 64 * j < ncols) F[(int64_t)g * ncols + c0 + 64 * j] = acc[j];
  }
}

// ---------------------------------------------------- several right-hand sides
//
// Aggregation of groups of few rows for 2 to 4 right-hand sides (RB columns held, nr of them
// valid): a thread walks all rows of two columns.  Such a group's output is as long as its
// input, and the matrix cores' tiles store a quarter of a line at a time: 200 groups of 8 rows
// and 5700 columns, 2 and 4 right-hand sides, complex128 30 and 42 us, 59 with those tiles;
// complex64 17 and 25 us, 33.  32 rows: complex128 124 and 138 us, 112 and 120 with the tiles;
// complex64 51 and 66, 53 and 56 (3000 groups of 40 rows and 196 columns, 2 right-hand sides:
// 40, 47; of 20 rows, complex128, 3: 41, 53).  Rows of few columns leave most of its threads
// idle (20000 groups of 9 rows and 30 columns, complex64, 3 right-hand sides: 64, 36).
template <typename T>
bool few_rows(int64_t n_rows, int n_groups, int ncols, int nrhs) {
  const int rows = sizeof(T) == 8 ? 24 : (nrhs == 2 ? 40 : 20);
  return nrhs <= 4 && ncols > 128 && n_rows <= (int64_t)rows * n_groups;
}
constexpr int kFewCols = 2;  // columns per thread
template <typename T, int RB>
__global__ __launch_bounds__(kThreads) void dense_agg_few_kernel(const typename Tr<T>::c* __restrict__ A,
                                                                 const DenseGroup* __restrict__ groups, int n_chunks,
                                                                 int ncols, int nrhs,
                                                                 const typename Tr<T>::c* __restrict__ x,
                                                                 typename Tr<T>::c* __restrict__ F) {
  using C = typename Tr<T>::c;
  constexpr int U = RB == 4 ? 2 : 4;  // rows in flight
  const int g = blockIdx.x / n_chunks;
  const int c0 = (blockIdx.x - g * n_chunks) * kThreads * kFewCols + threadIdx.x;
  const DenseGroup grp = groups[g];
  C acc[kFewCols][RB];
  int off[kFewCols];
#pragma unroll
  for (int j = 0; j < kFewCols; ++j) {
    off[j] = min(c0 + kThreads * j, ncols - 1);  // (columns past the end are not stored)
#pragma unroll
    for (int r = 0; r < RB; ++r) acc[j][r] = czero<C>();
  }
  const C* base = A + grp.row0 * ncols;
  const C* xb = x + grp.row0 * nrhs;
  auto rows = [&](int n, auto count) {
    C a[count][kFewCols];
#pragma unroll
    for (int u = 0; u < count; ++u)
#pragma unroll
      for (int j = 0; j < kFewCols; ++j) a[u][j] = base[(int64_t)(n + u) * ncols + off[j]];
#pragma unroll
    for (int u = 0; u < count; ++u)
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const C xn = r < nrhs ? xb[(int64_t)(n + u) * nrhs + r] : czero<C>();
#pragma unroll
        for (int j = 0; j < kFewCols; ++j) cfma(acc[j][r], a[u][j], xn);
      }
  };
  int n = 0;
  for (; n + U <= grp.nb; n += U) rows(n, std::integral_constant<int, U>{});
  for (; n < grp.nb; ++n) rows(n, std::integral_constant<int, 1>{});
#pragma unroll
  for (int j = 0; j < kFewCols; ++j) {
    if (c0 + kThreads * j >= ncols) continue;
    C* out = F + ((int64_t)g * ncols + c0 + kThreads * j) * nrhs;
#pragma unroll
    for (int r = 0; r < RB; ++r)
      if (r < nrhs) out[r] = acc[j][r];
  }
}

// FP32 and FP64 matrix instructions of 16 x 16 x 4: lane l feeds row (column) l % 16 and
// k = l / 16 of A (B); register i of lane l holds column l % 16 of row 4 (l / 16) + i
// (FP32) or 4 i + l / 16 (FP64).  Column 2 r + q of B is part q (real, imaginary) of
// right-hand side r, which is how a vector stores its values, so a lane reads one real
// number and a wavefront whole lines.  A complex product takes two instructions, one for
// each part of A:
//   aggregation    Re A [Re x, Im x]  +  Im A [-Im x, Re x]
//   disaggregation Re A [Re G, Im G]  +  Im A [ Im G, -Re G]   (conj A)
// whose second operand is the neighbouring lane's value, negated in one parity.  Columns
// past the last right-hand side read a clamped one and are not stored.  200 groups of 232
// rows and 2450 columns, complex128, 8 right-hand sides, both stages: 745 us (5.0 TB/s);
// 940 us with the products on the vector units, whose 64 sums a thread left two wavefronts
// a SIMD to hide the loads.
template <typename T>
struct DenseMfma;
template <>
struct DenseMfma<float> {
  typedef float acc __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc mul(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int i, int g) { return 4 * g + i; }
};
template <>
struct DenseMfma<double> {
  typedef double acc __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc mul(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int i, int g) { return 4 * i + g; }
};

// The neighbouring lane's value (lane l ^ 1).
__device__ __forceinline__ uint32_t other_lane(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true);
}
__device__ __forceinline__ float other_part(float v) { return __uint_as_float(other_lane(__float_as_uint(v))); }
__device__ __forceinline__ double other_part(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = other_lane((uint32_t)u), hi = other_lane((uint32_t)(u >> 32));
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Aggregation: a workgroup takes 16 MB columns of a group for up to 8 right-hand sides; its
// wavefronts take the rows in steps of 4, in turn, and meet in LDS.
template <typename T>
__global__ __launch_bounds__(kThreads) void dense_agg_mfma_kernel(const typename Tr<T>::c* __restrict__ A,
                                                                  const DenseGroup* __restrict__ groups, int n_chunks,
                                                                  int ncols, int nrhs,
                                                                  const typename Tr<T>::c* __restrict__ x,
                                                                  typename Tr<T>::c* __restrict__ F) {
  using C = typename Tr<T>::c;
  using Acc = typename DenseMfma<T>::acc;
  constexpr int MB = 4;
  constexpr int U = 2;  // steps in flight
  __shared__ T sum[kWaves - 1][MB][4][64];
  const int g = blockIdx.x / n_chunks;
  const int lane = threadIdx.x & 63, li = lane & 15, kg = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int c0 = (blockIdx.x - g * n_chunks) * 16 * MB;
  const int r0 = blockIdx.y * 8, nr = min(8, nrhs - r0);
  const DenseGroup grp = groups[g];
  const int part = min(li, 2 * nr - 1);
  const C* base = A + grp.row0 * ncols;
  const T* xb = reinterpret_cast<const T*>(x + grp.row0 * nrhs + r0) + part;
  int off[MB];
#pragma unroll
  for (int m = 0; m < MB; ++m) off[m] = min(c0 + 16 * m + li, ncols - 1);
  Acc acc[MB];
#pragma unroll
  for (int m = 0; m < MB; ++m) acc[m] = Acc{0, 0, 0, 0};
  for (int n0 = 4 * w; n0 < grp.nb; n0 += 4 * kWaves * U) {
    C a[U][MB];
    T b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int n = n0 + 4 * kWaves * u + kg, nc = min(n, grp.nb - 1);
#pragma unroll
      for (int m = 0; m < MB; ++m) a[u][m] = base[(int64_t)nc * ncols + off[m]];
      b[u] = xb[(int64_t)nc * 2 * nrhs];
      if (n >= grp.nb) {
        b[u] = T(0);
#pragma unroll
        for (int m = 0; m < MB; ++m) a[u][m] = czero<C>();
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const T o = other_part(b[u]), b2 = li & 1 ? o : -o;
#pragma unroll
      for (int m = 0; m < MB; ++m) acc[m] = DenseMfma<T>::mul(a[u][m].x, b[u], acc[m]);
#pragma unroll
      for (int m = 0; m < MB; ++m) acc[m] = DenseMfma<T>::mul(a[u][m].y, b2, acc[m]);
    }
  }
  if (w > 0) {
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) sum[w - 1][m][i][lane] = acc[m][i];
  }
  __syncthreads();
  if (w > 0 || li >= 2 * nr) return;
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      T v = acc[m][i];
#pragma unroll
      for (int k = 0; k < kWaves - 1; ++k) v += sum[k][m][i][lane];
      const int c = c0 + 16 * m + DenseMfma<T>::row(i, kg);
      if (c < ncols) reinterpret_cast<T*>(F + ((int64_t)g * ncols + c) * nrhs + r0)[li] = v;
    }
}

// A 16-byte pack of a row of A or an element of it, read at the element's alignment.
template <typename T>
struct RowPack;
template <>
struct RowPack<float> {
  typedef float v __attribute__((ext_vector_type(4), aligned(8)));
};
template <>
struct RowPack<double> {
  typedef double v __attribute__((ext_vector_type(2), aligned(16)));
};

// Disaggregation: a workgroup takes a block of up to 16 rows of one group for up to 8
// right-hand sides; its eight wavefronts take chunks of columns in turn and meet in LDS.  The
// plan orders the blocks so that each XCD works on a few groups at a time, whose G then stays
// in its L2 (it is read once per block, half the bytes of A's).
//
// Lane (li, kg) reads kPacks packs of 16 bytes of row li a chunk, neighbouring kg's adjacent:
// 64 bytes of a row an instruction.  Both A and B take the packs' columns as the K index, so
// their order is free.  Each pack, wavefront and part of A has its own accumulators, 64 in
// all, that meet in a tree: a chain is as long as that of 64 lanes which share a row, and so
// is its rounding error.  8 right-hand sides, complex64 / complex128: 24 groups of mean 909
// rows and 5700 columns take 228 / 391 us (4.4 / 5.1 TB/s), two such groups 27 / 44 us; with
// one wavefront a block, reads of one element and one accumulator a part they took 762 / 400
// and 473 / 211 us, and the error was five to ten times as large.
constexpr int kDisThreads = 512;
constexpr int kDisWaves = kDisThreads / 64;
template <typename T>
__global__ __launch_bounds__(kDisThreads) void dense_disagg_mfma_kernel(const typename Tr<T>::c* __restrict__ A,
                                                                        const DenseBlock* __restrict__ blocks,
                                                                        int ncols, int nrhs,
                                                                        const typename Tr<T>::c* __restrict__ Gin,
                                                                        typename Tr<T>::c* __restrict__ V) {
  using C = typename Tr<T>::c;
  using Acc = typename DenseMfma<T>::acc;
  using Pack = typename RowPack<T>::v;
  constexpr int E = Tr<T>::E;
  constexpr int kPacks = 4;
  constexpr int kChunk = 4 * E * kPacks;  // columns of a wavefront's step
  __shared__ T sum[kDisWaves - 1][4][64];
  const int lane = threadIdx.x & 63, li = lane & 15, kg = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const DenseBlock b = blocks[blockIdx.x];
  const int r0 = blockIdx.y * 8, nr = min(8, nrhs - r0);
  const C* row = A + (b.row0 + min(li, b.rows - 1)) * ncols;
  const T* gv = reinterpret_cast<const T*>(Gin + (int64_t)b.group * ncols * nrhs + r0) + min(li, 2 * nr - 1);
  Acc acc[kPacks][2];
#pragma unroll
  for (int q = 0; q < kPacks; ++q) acc[q][0] = acc[q][1] = Acc{0, 0, 0, 0};
  // (ncols counts both polarisations, so it is even and a complex64 pack is whole or absent)
  auto chunk = [&](int c0, auto tail) {
    Pack a[kPacks];
    T g[kPacks][E];
#pragma unroll
    for (int q = 0; q < kPacks; ++q) {
      const int c = c0 + (4 * q + kg) * E, cc = tail ? min(c, ncols - E) : c;
      a[q] = *reinterpret_cast<const Pack*>(row + cc);
#pragma unroll
      for (int e = 0; e < E; ++e) g[q][e] = gv[(int64_t)(cc + e) * 2 * nrhs];
      if (tail && c >= ncols) {
#pragma unroll
        for (int e = 0; e < E; ++e) a[q][2 * e] = a[q][2 * e + 1] = g[q][e] = T(0);
      }
    }
#pragma unroll
    for (int e = 0; e < E; ++e)
#pragma unroll
      for (int q = 0; q < kPacks; ++q) {
        const T o = other_part(g[q][e]), g2 = li & 1 ? -o : o;
        acc[q][0] = DenseMfma<T>::mul(a[q][2 * e], g[q][e], acc[q][0]);
        acc[q][1] = DenseMfma<T>::mul(a[q][2 * e + 1], g2, acc[q][1]);
      }
  };
  int c0 = kChunk * w;
  for (; c0 + kChunk <= ncols; c0 += kChunk * kDisWaves) chunk(c0, std::false_type{});
  if (c0 < ncols) chunk(c0, std::true_type{});
  T v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    v[i] = ((acc[0][0][i] + acc[0][1][i]) + (acc[1][0][i] + acc[1][1][i])) +
           ((acc[2][0][i] + acc[2][1][i]) + (acc[3][0][i] + acc[3][1][i]));
  if (w > 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) sum[w - 1][i][lane] = v[i];
  }
  __syncthreads();
  if (w > 0 || li >= 2 * nr) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = DenseMfma<T>::row(i, kg);
    const T s = ((v[i] + sum[0][i][lane]) + (sum[1][i][lane] + sum[2][i][lane])) +
                ((sum[3][i][lane] + sum[4][i][lane]) + (sum[5][i][lane] + sum[6][i][lane]));
    if (m < b.rows) reinterpret_cast<T*>(V + (b.row0 + m) * nrhs + r0)[li] = s;
  }
}

// Disaggregation with one right-hand side: a wavefront per row, four columns in
// flight per lane, butterfly sum.
template <typename T>
__global__ __launch_bounds__(kThreads) void dense_disagg_kernel(const typename Tr<T>::c* __restrict__ A,
                                                                const int64_t* __restrict__ offsets,
                                                                int n_groups, int64_t n_rows, int ncols,
                                                                const typename Tr<T>::c* __restrict__ Gin,
                                                                typename Tr<T>::c* __restrict__ V) {
  using C = typename Tr<T>::c;
  constexpr int U = 4;  // columns in flight per lane
  const int lane = threadIdx.x & 63;
  const int64_t n = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  if (n >= n_rows) return;  // no barrier below
  // group of row n: largest g with offsets[g] <= n
  int lo = 0, hi = n_groups;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (offsets[mid] <= n) lo = mid; else hi = mid;
  }
  const C* row = A + n * ncols;
  const C* gv = Gin + (int64_t)lo * ncols;
  C acc[U];
#pragma unroll
  for (int u = 0; u < U; ++u) acc[u] = czero<C>();
  int c = lane;
  for (; c + 64 * (U - 1) < ncols; c += 64 * U) {
    C a[U];
#pragma unroll
    for (int u = 0; u < U; ++u) a[u] = row[c + 64 * u];
#pragma unroll
    for (int u = 0; u < U; ++u) cfma_conj(acc[u], a[u], gv[c + 64 * u]);
  }
  for (; c < ncols; c += 64) cfma_conj(acc[0], row[c], gv[c]);
  C s = acc[0];
#pragma unroll
  for (int u = 1; u < U; ++u) {
    s.x += acc[u].x;
    s.y += acc[u].y;
  }
  s = wave_sum(s);
  if (lane == 0) V[n] = s;
}

}  // namespace

// Workgroups of one launch along x (a grid holds fewer than 2^32 threads); layouts of more run
// as several launches.
constexpr int kMaxGrid = 1 << 22;

template <typename T>
hipError_t launch_dense_agg(const void* A, const DenseGroup* groups, int n_groups, int64_t n_rows, int ncols, int nrhs,
                            const void* x, void* F, hipStream_t s) {
  using C = typename Tr<T>::c;
  const bool few = few_rows<T>(n_rows, n_groups, ncols, nrhs);
  const int cols = nrhs == 1 ? 128 * Tr<T>::E : (few ? kThreads * kFewCols : 64);  // of a workgroup
  const int n_chunks = (ncols + cols - 1) / cols, step = std::max(1, kMaxGrid / n_chunks);
  const C* a = static_cast<const C*>(A);
  const C* xv = static_cast<const C*>(x);
  hipError_t e = hipSuccess;
  for (int64_t g0 = 0; g0 < n_groups && e == hipSuccess; g0 += step) {
    const unsigned blocks = (unsigned)std::min<int64_t>(step, n_groups - g0) * n_chunks;
    C* f = static_cast<C*>(F) + g0 * ncols * nrhs;
    if (nrhs == 1)
      hipLaunchKernelGGL(dense_agg_kernel<T>, dim3(blocks), dim3(kThreads), 0, s, a, groups + g0, n_chunks, ncols, xv, f);
    else if (few)
      hipLaunchKernelGGL((nrhs == 2 ? dense_agg_few_kernel<T, 2> : dense_agg_few_kernel<T, 4>), dim3(blocks),
                         dim3(kThreads), 0, s, a, groups + g0, n_chunks, ncols, nrhs, xv, f);
    else
      hipLaunchKernelGGL(dense_agg_mfma_kernel<T>, dim3(blocks, (nrhs + 7) / 8), dim3(kThreads), 0, s, a, groups + g0,
                         n_chunks, ncols, nrhs, xv, f);
    e = hipGetLastError();
  }
  return e;
}

template <typename T>
hipError_t launch_dense_disagg(const void* A, const int64_t* offsets, int n_groups, int64_t n_rows,
                               const DenseBlock* row_blocks, int n_blocks, int ncols, int nrhs, const void* G,
                               void* V, hipStream_t s) {
  using C = typename Tr<T>::c;
  if (n_rows == 0) return hipSuccess;
  if (nrhs == 1) {
    const int64_t blocks = (n_rows + kWaves - 1) / kWaves;
    hipLaunchKernelGGL((dense_disagg_kernel<T>), dim3((unsigned)blocks), dim3(kThreads), 0, s,
                       static_cast<const C*>(A), offsets, n_groups, n_rows, ncols, static_cast<const C*>(G),
                       static_cast<C*>(V));
    return hipGetLastError();
  }
  if (n_blocks <= 0 || row_blocks == nullptr) return hipErrorInvalidValue;
  hipError_t e = hipSuccess;
  for (int64_t b0 = 0; b0 < n_blocks && e == hipSuccess; b0 += kMaxGrid) {
    const unsigned blocks = (unsigned)std::min<int64_t>(kMaxGrid, n_blocks - b0);
    hipLaunchKernelGGL((dense_disagg_mfma_kernel<T>), dim3(blocks, (nrhs + 7) / 8), dim3(kDisThreads), 0, s,
                       static_cast<const C*>(A), row_blocks + b0, ncols, nrhs, static_cast<const C*>(G),
                       static_cast<C*>(V));
    e = hipGetLastError();
  }
  return e;
}

template hipError_t launch_dense_agg<float>(const void*, const DenseGroup*, int, int64_t, int, int, const void*,
                                            void*, hipStream_t);
template hipError_t launch_dense_agg<double>(const void*, const DenseGroup*, int, int64_t, int, int, const void*,
                                             void*, hipStream_t);
template hipError_t launch_dense_disagg<float>(const void*, const int64_t*, int, int64_t, const DenseBlock*, int,
                                               int, int, const void*, void*, hipStream_t);
template hipError_t launch_dense_disagg<double>(const void*, const int64_t*, int, int64_t, const DenseBlock*, int,
                                                int, int, const void*, void*, hipStream_t);

}  // namespace tuckfmm
