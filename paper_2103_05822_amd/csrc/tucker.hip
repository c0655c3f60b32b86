// Tucker-format aggregation and disaggregation (Section II.C, Figs. 2(b) and 3(b)) for one
// to a few right-hand sides.
//
// One workgroup of NT = 64, 128, 256 or 512 threads per (group, polarisation) work item and
// block of right-hand sides, NT chosen from the mean item size and, for several right-hand
// sides, the longest row.  Work lists are sorted by decreasing cost
// (longest-processing-time order).  In layouts of few items, large items run as blocks of
// their r_beta rows (work units) whose partial sums a finishing kernel adds in block order.
// Per item (g, alpha), the angular order chosen on the host:
//   S[a,c] = sum U^theta[i][a] U^phi[j][c] conj(G[i,j])    angular phase, matrix cores
//   for every row b of U^beta^T and the core:
//     y[b] = sum_n U^beta[n][b] x[n],   t[q] += core[b][q] y[b]
//     s[b] = sum_q core[b][q] S[q],     v[n] += U^beta[n][b] s[b]
//   F[i,j] = sum U^theta[i][a] U^phi[j][c] t[a, c]         angular phase, matrix cores
//   V[n]  += conj(v[n])   atomically onto a zeroed V: each entry receives exactly two
//            additions onto zero, one per polarisation, which commute exactly, so the
//            result does not depend on which polarisation finishes first.
// The sweep over the rows reads each factor once for both stages (the row-streaming kernels
// below).  Layouts with rows too long for its registers run on the general kernel, which
// reads the factors once per stage and keeps every vector in LDS.
//
// One-right-hand-side pass on an MI355X, before (one read of the factors per stage, angular
// products on the vector units) and now: 4000 items of mean 15k elements, complex64, 231 and
// 128 us (510 MB: 4.0 TB/s); 512 items of mean 259k 398 and 229 us (1.2 GB: 5.2 TB/s); both
// stages alone, complex128, 800 items of mean 58k 472 and 307 us (1.6 GB: 5.2 TB/s).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "cplx.hpp"
#include "kernels.hpp"

namespace tuckfmm {

// This file is compiled twice, for each of the two element types (see tucker_f64.hip).
#ifdef TUCKFMM_STREAM_F64
using Real = double;
#else
using Real = float;
#endif

namespace {

// The general kernel's workgroup size.
constexpr int kGenThreads = 512;
constexpr int kColPacks = 2;  // column packs per thread per chunk in the axpy stages
// U^beta^T and the core are read once per call: the 256- and 512-thread kernels, which large
// items take, load them non-temporally, so that these streams don't displace x, G, V and
// the work tables in the caches (5-7% on boxes of 2 wavelengths and more; on small items it
// cost 4%).  The general kernel's loads:
template <typename P>
struct NtVec;
template <>
struct NtVec<float4> {
  typedef float v __attribute__((ext_vector_type(4)));
};
template <>
struct NtVec<double2> {
  typedef double v __attribute__((ext_vector_type(2)));
};
template <typename P>
__device__ __forceinline__ P ldnt(const P* p) {
  const auto v = __builtin_nontemporal_load(reinterpret_cast<const typename NtVec<P>::v*>(p));
  P o;
  __builtin_memcpy(&o, &v, sizeof(P));
  return o;
}

// LDS regions of the general kernel (complex elements).
// Aggregation:    r1 = x (n_beta), later t (r_theta r_phi);  r2 = y (r_beta), later
//                 the angular intermediate.
// Disaggregation: s1 = angular intermediate, S (r_theta r_phi), s (r_beta).
template <typename T>
struct Lds {
  int r1, r2, s1, s2, s3;
  __host__ __device__ explicit Lds(const TuckMax& mx) {
    constexpr int E = Tr<T>::E;
    r1 = round_up(max(round_up(mx.nb, E), round_up(mx.q, E)), 2);
    r2 = round_up(max(mx.rb, mx.t3), 2);
    s1 = round_up(mx.t3, 2);
    s2 = round_up(round_up(mx.q, E), 2);
    s3 = round_up(mx.rb, 2);
  }
  __host__ __device__ size_t agg_bytes() const { return size_t(r1 + r2) * sizeof(typename Tr<T>::c); }
  __host__ __device__ size_t dis_bytes() const { return size_t(s1 + s2 + s3) * sizeof(typename Tr<T>::c); }
  __host__ __device__ size_t bytes() const { return agg_bytes() > dis_bytes() ? agg_bytes() : dis_bytes(); }
};

// Short rows (npk <= 32 packs): the wavefront splits into 64 / S segments of S lanes,
// S the smallest power of two >= npk, and each segment takes a row, four rows per
// segment in flight, so a wavefront works on 4 * 64 / S rows at once instead of four
// mostly idle ones; the segment's sum is a butterfly over its S lanes.
template <typename T>
__device__ __forceinline__ void wave_rowdots_short(const typename Tr<T>::c* rows, int ld, int first, int last,
                                                   int step, const typename Tr<T>::pack* vec, int npk,
                                                   typename Tr<T>::c* out, int lane) {
  using C = typename Tr<T>::c;
  using P = typename Tr<T>::pack;
  int S = 1;
  while (S < npk) S <<= 1;
  const int G = 64 / S;             // segments (rows) per wavefront
  const int seg = lane / S, sl = lane - seg * S;
  const bool act = sl < npk;
  const P v = act ? vec[sl] : pzero<P>();
  for (int j0 = 0; first + step * j0 < last; j0 += 4 * G) {
    P u[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int b = first + step * (j0 + G * i + seg);
      u[i] = (act && b < last) ? ldnt(reinterpret_cast<const P*>(rows + (int64_t)b * ld) + sl) : pzero<P>();
    }
    C a[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      a[i] = czero<C>();
      pdot(a[i], u[i], v);
    }
    for (int o = S >> 1; o > 0; o >>= 1) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a[i].x += __shfl_xor(a[i].x, o, 64);
        a[i].y += __shfl_xor(a[i].y, o, 64);
      }
    }
    if (sl == 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int b = first + step * (j0 + G * i + seg);
        if (b < last) out[b] = a[i];
      }
    }
  }
}

// out[b] = sum_k rows[b][k] * vec[k] for b = first, first + step, ... < last, one
// wavefront per row.  Rows are 16-byte aligned with npk packs each; vec is an LDS
// pack array.  Four rows at a time, two packs per row per iteration: eight 16-byte
// loads in flight per lane.  Rows of at most 32 packs take the segmented form above.
template <typename T>
__device__ __forceinline__ void wave_rowdots(const typename Tr<T>::c* rows, int ld, int first, int last,
                                             int step, const typename Tr<T>::pack* vec, int npk,
                                             typename Tr<T>::c* out, int lane) {
  using C = typename Tr<T>::c;
  using P = typename Tr<T>::pack;
  if (npk <= 32) {
    wave_rowdots_short<T>(rows, ld, first, last, step, vec, npk, out, lane);
    return;
  }
  int b = first;
  for (; b + 3 * step < last; b += 4 * step) {
    const P* r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = reinterpret_cast<const P*>(rows + (int64_t)(b + i * step) * ld);
    C a[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = czero<C>();
    int p = lane;
    for (; p + 64 < npk; p += 128) {
      P u[4], w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        u[i] = ldnt(r[i] + p);
        w[i] = ldnt(r[i] + p + 64);
      }
      const P v0 = vec[p], v1 = vec[p + 64];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        pdot(a[i], u[i], v0);
        pdot(a[i], w[i], v1);
      }
    }
    if (p < npk) {
      P u[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) u[i] = ldnt(r[i] + p);
      const P v0 = vec[p];
#pragma unroll
      for (int i = 0; i < 4; ++i) pdot(a[i], u[i], v0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = wave_sum(a[i]);
    if (lane == 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) out[b + i * step] = a[i];
    }
  }
  for (; b < last; b += step) {
    const P* r0 = reinterpret_cast<const P*>(rows + (int64_t)b * ld);
    C a0 = czero<C>(), a1 = czero<C>();
    int p = lane;
    for (; p + 64 < npk; p += 128) {
      const P u0 = ldnt(r0 + p), u1 = ldnt(r0 + p + 64);
      pdot(a0, u0, vec[p]);
      pdot(a1, u1, vec[p + 64]);
    }
    if (p < npk) pdot(a0, ldnt(r0 + p), vec[p]);
    a0.x += a1.x;
    a0.y += a1.y;
    a0 = wave_sum(a0);
    if (lane == 0) out[b] = a0;
  }
}

// acc[j] (column packs base + tid + NT j) += sum_b rows[b][.] * coef[b];
// four rows per iteration.
template <typename T, int NT>
__device__ __forceinline__ void block_colaxpy(const typename Tr<T>::c* rows, int ld, int nrows,
                                              const typename Tr<T>::c* coef, int npk, int base, int tid,
                                              typename Tr<T>::pack (&acc)[kColPacks]) {
  using C = typename Tr<T>::c;
  using P = typename Tr<T>::pack;
  const int p0 = base + tid;
  bool in[kColPacks];
#pragma unroll
  for (int j = 0; j < kColPacks; ++j) in[j] = p0 + NT * j < npk;
  int b = 0;
  for (; b + 3 < nrows; b += 4) {
    P u[4][kColPacks];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const P* r = reinterpret_cast<const P*>(rows + (int64_t)(b + i) * ld);
#pragma unroll
      for (int j = 0; j < kColPacks; ++j) u[i][j] = in[j] ? ldnt(r + p0 + NT * j) : pzero<P>();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const C c = coef[b + i];
#pragma unroll
      for (int j = 0; j < kColPacks; ++j) paxpy(acc[j], u[i][j], c);
    }
  }
  for (; b < nrows; ++b) {
    const P* r = reinterpret_cast<const P*>(rows + (int64_t)b * ld);
    const C c = coef[b];
#pragma unroll
    for (int j = 0; j < kColPacks; ++j)
      if (in[j]) paxpy(acc[j], ldnt(r + p0 + NT * j), c);
  }
}

// FP32 and FP64 matrix instructions of 16 x 16 x 4: lane l feeds row (column) l % 16 and
// k = l / 16 of A (B); register i of lane l holds column l % 16 of row 4 (l / 16) + i
// (FP32) or 4 i + l / 16 (FP64).
template <typename T>
struct Mfma;
template <>
struct Mfma<float> {
  typedef float acc __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc mul(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int i, int g) { return 4 * g + i; }
};
template <>
struct Mfma<double> {
  typedef double acc __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc mul(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int i, int g) { return 4 * i + g; }
};

// out(m, n) = sum_k a(m, k) * b(k, n) for m < M, n < N: a small complex product of the
// angular phases, computed by the whole workgroup on the matrix cores in tiles of
// 16 x 16 values, tiles over wavefronts.  Four real products make a complex one; a step
// of 4 K values reads one value of each operand per lane.  (On the vector units, with
// four rows per thread, the products read five LDS values per four complex multiply-adds
// and were bound by that.)
template <typename T, int NT, class FA, class FB, class FO>
__device__ __forceinline__ void tile_product(int M, int N, int K, FA a, FB b, FO out, int tid) {
  using C = typename Tr<T>::c;
  using Acc = typename Mfma<T>::acc;
  constexpr int KU = 4;  // steps whose operands are loaded before their products
  const int lane = tid & 63, li = lane & 15, g = lane >> 4;
  const int mt = (M + 15) >> 4, tiles = mt * ((N + 15) >> 4);
  for (int t = __builtin_amdgcn_readfirstlane(tid >> 6); t < tiles; t += NT / 64) {
    const int n0 = t / mt * 16, m0 = (t - t / mt * mt) * 16;
    const int m = min(m0 + li, M - 1), n = min(n0 + li, N - 1);  // (rows past the end are not stored)
    Acc re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
    for (int k0 = 0; k0 < K; k0 += 4 * KU) {
      C av[KU], bv[KU];
#pragma unroll
      for (int j = 0; j < KU; ++j) {
        const int k = k0 + 4 * j + g, kc = min(k, K - 1);
        av[j] = a(m, kc);
        bv[j] = b(kc, n);
        if (k >= K) av[j] = bv[j] = czero<C>();
      }
#pragma unroll
      for (int j = 0; j < KU; ++j) {
        if (k0 + 4 * j >= K) break;
        re = Mfma<T>::mul(av[j].x, bv[j].x, re);
        im = Mfma<T>::mul(av[j].x, bv[j].y, im);
        re = Mfma<T>::mul(-av[j].y, bv[j].y, re);
        im = Mfma<T>::mul(av[j].y, bv[j].x, im);
      }
    }
    if (n0 + li < N) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = m0 + Mfma<T>::row(i, g);
        if (row < M) out(row, n0 + li, C{re[i], im[i]});
      }
    }
  }
}

__device__ __forceinline__ void atomic_add_c(float2* p, float2 v) {
  atomicAdd(&p->x, v.x);
  atomicAdd(&p->y, v.y);
}
__device__ __forceinline__ void atomic_add_c(double2* p, double2 v) {
  atomicAdd(&p->x, v.x);
  atomicAdd(&p->y, v.y);
}

// ------------------------------------------------------------------ aggregation

// Streaming phase over rows [b0, b1) of U^beta^T and the core: y = U^beta^T x
// (row-dots), then t = core^T y (column axpy) written as packs to `t_out` -- LDS for
// a whole item, the unit's partial-sum block in global memory for a row block of a
// split item.  t[q], q = theta' r_phi + phi'.
template <typename T, int NT>
__device__ __forceinline__ void agg_stream(const typename Tr<T>::c* __restrict__ fac, const TuckItem& it,
                                           const Lds<T>& L, unsigned char* smem, int nrhs, int r,
                                           const typename Tr<T>::c* __restrict__ x, int b0, int b1,
                                           typename Tr<T>::c* t_out) {
  using C = typename Tr<T>::c;
  using P = typename Tr<T>::pack;
  constexpr int E = Tr<T>::E;
  C* xs = reinterpret_cast<C*>(smem);
  C* ys = xs + L.r1;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nb = it.nb, Q = it.rt * it.rp;
  const int nbp = round_up(nb, E);

  // x of the group into LDS (zero padded to whole packs)
  for (int n = tid; n < nbp; n += NT) xs[n] = n < nb ? x[(it.row0 + n) * nrhs + r] : czero<C>();
  __syncthreads();

  // y = U^beta^T x (rows b0 .. b1 - 1)
  wave_rowdots<T>(fac + it.off_ubt, it.ld_ub, b0 + wave, b1, (NT / 64), reinterpret_cast<const P*>(xs), nbp / E,
                  ys, lane);
  __syncthreads();

  // t = core^T y over the same rows; t_out may alias x, which is no longer read
  const int qpk = round_up(Q, E) / E;
  for (int base = 0; base < qpk; base += NT * kColPacks) {
    P acc[kColPacks];
#pragma unroll
    for (int j = 0; j < kColPacks; ++j) acc[j] = pzero<P>();
    block_colaxpy<T, NT>(fac + it.off_core + (int64_t)b0 * it.ld_c, it.ld_c, b1 - b0, ys + b0, qpk, base, tid,
                         acc);
#pragma unroll
    for (int j = 0; j < kColPacks; ++j) {
      const int p = base + tid + NT * j;
      if (p < qpk) reinterpret_cast<P*>(t_out)[p] = acc[j];
    }
  }
}

// The angular factors where the angular phases read them: U^theta [n_theta][r_theta] and
// U^phi [n_phi][r_phi], in global memory, or staged in LDS with odd row strides (which
// spread the matrix instructions' operand reads over the banks).  The address space is in
// the type, so that neither becomes a flat access.
template <typename C>
struct GlobalAngular {
  const C* __restrict__ ut;
  const C* __restrict__ up;
  int ldt, ldp;
  __device__ __forceinline__ C t(int i, int a) const { return ut[i * ldt + a]; }
  __device__ __forceinline__ C p(int j, int c) const { return up[j * ldp + c]; }
};
template <typename C>
struct LdsAngular {
  typedef const C __attribute__((address_space(3))) * Ptr;
  Ptr ut, up;
  int ldt, ldp;
  __device__ __forceinline__ C t(int i, int a) const { return lds_value(ut + i * ldt + a); }
  __device__ __forceinline__ C p(int j, int c) const { return lds_value(up + j * ldp + c); }
  static __device__ __forceinline__ C lds_value(Ptr q) {
    typedef decltype(C{}.x) R2 __attribute__((ext_vector_type(2)));
    const R2 v = *(const R2 __attribute__((address_space(3))) *)q;
    return C{v.x, v.y};
  }
};
template <typename T>
__device__ __forceinline__ GlobalAngular<typename Tr<T>::c> global_angular(const typename Tr<T>::c* fac,
                                                                            const TuckItem& it) {
  return {fac + it.off_ut, fac + it.off_up, it.rt, it.rp};
}
// Staged by stage_in at `us` (an LDS address).
template <typename T>
__device__ __forceinline__ LdsAngular<typename Tr<T>::c> staged_angular(const typename Tr<T>::c* us,
                                                                         const TuckItem& it, int n_theta) {
  using P = typename LdsAngular<typename Tr<T>::c>::Ptr;
  return {(P)us, (P)(us + round_up(n_theta * (it.rt | 1), 2)), it.rt | 1, it.rp | 1};
}

// Angular phase of the aggregation: F = U^theta t U^phi^T from t in LDS (`ts`), with the
// intermediate at `t3`.
template <typename T, int NT, class FA>
__device__ __forceinline__ void agg_angular(const TuckItem& it, const FA& f, typename Tr<T>::c* t3,
                                            const typename Tr<T>::c* ts, int n_theta, int n_phi, int nrhs, int r,
                                            typename Tr<T>::c* __restrict__ F) {
  using C = typename Tr<T>::c;
  const int tid = threadIdx.x;
  const int rt = it.rt, rp = it.rp;
  const int ndir = n_theta * n_phi;
  C* Fo = F + ((int64_t)it.frow * ndir) * nrhs + r;
  if (it.ident) {  // truncated-SVD item: t already holds the directions
    for (int i = tid; i < ndir; i += NT) Fo[(int64_t)i * nrhs] = ts[i];
    return;
  }
  if (it.theta_first) {
    // t3[i][c] = sum_a U^theta[i][a] t[a][c]           (n_theta x r_phi)
    tile_product<T, NT>(
        n_theta, rp, rt, [&](int i, int a) { return f.t(i, a); },
        [&](int a, int c) { return ts[a * rp + c]; }, [&](int i, int c, C v) { t3[i * rp + c] = v; }, tid);
    __syncthreads();
    // F[i][j] = sum_c t3[i][c] U^phi[j][c]
    tile_product<T, NT>(
        n_theta, n_phi, rp, [&](int i, int c) { return t3[i * rp + c]; },
        [&](int c, int j) { return f.p(j, c); },
        [&](int i, int j, C v) { Fo[(int64_t)(i * n_phi + j) * nrhs] = v; }, tid);
  } else {
    // t3[a][j] = sum_c t[a][c] U^phi[j][c]             (r_theta x n_phi)
    tile_product<T, NT>(
        rt, n_phi, rp, [&](int a, int c) { return ts[a * rp + c]; },
        [&](int c, int j) { return f.p(j, c); }, [&](int a, int j, C v) { t3[a * n_phi + j] = v; }, tid);
    __syncthreads();
    // F[i][j] = sum_a U^theta[i][a] t3[a][j]
    tile_product<T, NT>(
        n_theta, n_phi, rt, [&](int i, int a) { return f.t(i, a); },
        [&](int a, int j) { return t3[a * n_phi + j]; },
        [&](int i, int j, C v) { Fo[(int64_t)(i * n_phi + j) * nrhs] = v; }, tid);
  }
}

// --------------------------------------------------------------- disaggregation

// Angular phase of the disaggregation: S = U^theta^T conj(G) U^phi, written with its pack
// padding to `S2` in LDS, with the intermediate at `s1`.  `gc(q)`: conj(G) of direction q.
template <typename T, int NT, class FA, class FG>
__device__ __forceinline__ void dis_angular(const TuckItem& it, const FA& f, typename Tr<T>::c* s1, int n_theta,
                                            int n_phi, FG gc, typename Tr<T>::c* S2) {
  using C = typename Tr<T>::c;
  const int tid = threadIdx.x;
  const int rt = it.rt, rp = it.rp, Q = rt * rp;
  // the angular order mirrors the aggregation choice
  if (it.ident) {  // truncated-SVD item: S2 is conj(G) itself
    for (int q = tid; q < Q; q += NT) S2[q] = gc(q);
  } else if (!it.theta_first) {
    // s1[a][j] = sum_i U^theta[i][a] conj(G[i][j])     (r_theta x n_phi)
    tile_product<T, NT>(
        rt, n_phi, n_theta, [&](int a, int i) { return f.t(i, a); },
        [&](int i, int j) { return gc(i * n_phi + j); }, [&](int a, int j, C v) { s1[a * n_phi + j] = v; }, tid);
    __syncthreads();
    // S[a][c] = sum_j s1[a][j] U^phi[j][c]
    tile_product<T, NT>(
        rt, rp, n_phi, [&](int a, int j) { return s1[a * n_phi + j]; },
        [&](int j, int c) { return f.p(j, c); }, [&](int a, int c, C v) { S2[a * rp + c] = v; }, tid);
  } else {
    // s1[i][c] = sum_j conj(G[i][j]) U^phi[j][c]       (n_theta x r_phi)
    tile_product<T, NT>(
        n_theta, rp, n_phi, [&](int i, int j) { return gc(i * n_phi + j); },
        [&](int j, int c) { return f.p(j, c); }, [&](int i, int c, C v) { s1[i * rp + c] = v; }, tid);
    __syncthreads();
    // S[a][c] = sum_i U^theta[i][a] s1[i][c]
    tile_product<T, NT>(
        rt, rp, n_theta, [&](int a, int i) { return f.t(i, a); },
        [&](int i, int c) { return s1[i * rp + c]; }, [&](int a, int c, C v) { S2[a * rp + c] = v; }, tid);
  }
  for (int o = Q + tid; o < round_up(Q, Tr<T>::E); o += NT) S2[o] = czero<C>();  // pack padding
}

// q / d for 0 <= q < 2^20 (LDS holds fewer values), `inv` = 1 / d rounded: the quotient of
// q + 1/2 is at least 1 / (2 d) from a whole number, more than the roundings of its size.
__device__ __forceinline__ int quot(int q, int d, float inv) { return d == 1 ? q : (int)(((float)q + 0.5f) * inv); }

// Copies parts of global memory to LDS with 64 bytes of loads in flight per thread, so
// that everything a unit needs before its sweep costs about one memory latency:
// x of the group (rows x0 ..; `nr` columns), conj(G) of the item's fibre and the angular
// factors (rows of odd stride).  Null destinations are left out.
template <typename T, int NT>
__device__ __forceinline__ void stage_in(const typename Tr<T>::c* fac, const TuckItem& it, int n_theta, int n_phi,
                                         int nrhs, const typename Tr<T>::c* x, int nr, typename Tr<T>::c* xs, int xrow,
                                         const typename Tr<T>::c* g, typename Tr<T>::c* gs, typename Tr<T>::c* us) {
  using C = typename Tr<T>::c;
  const int tid = threadIdx.x;
  const int rt = it.rt, rp = it.rp, ldt = rt | 1, ldp = rp | 1;
  const int n_x = x ? it.nb * nr : 0, n_g = gs ? n_theta * n_phi : 0, n_t = us ? n_theta * rt : 0,
            n_p = us ? n_phi * rp : 0;
  const int e1 = n_x + n_g, e2 = e1 + n_t, total = e2 + n_p;
  C* ups = us + round_up(n_theta * ldt, 2);
  const C* ut = fac + it.off_ut - e1;
  const C* up = fac + it.off_up - e2;
  const C* xg = x + it.row0 * nrhs;
  constexpr int U = 64 / sizeof(C);
  for (int i0 = tid; i0 < total; i0 += U * NT) {
    C v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = i0 + u * NT;
      if (e < total) {
        const int ex = quot(e, nr, 1.0f / nr);
        const C* src = e < n_x  ? xg + (int64_t)ex * nrhs + (e - ex * nr)
                       : e < e1 ? g + (int64_t)(e - n_x) * nrhs
                       : e < e2 ? ut + e
                                : up + e;
        v[u] = *src;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = i0 + u * NT;
      if (e < n_x) {
        const int ex = quot(e, nr, 1.0f / nr);
        xs[(e - ex * nr) * xrow + ex] = v[u];
      } else if (e < e1) {
        gs[e - n_x] = conjc(v[u]);
      } else if (e < e2) {
        const int q = e - e1, i = quot(q, rt, 1.0f / rt);
        us[i * ldt + (q - i * rt)] = v[u];
      } else if (e < total) {
        const int q = e - e2, j = quot(q, rp, 1.0f / rp);
        ups[j * ldp + (q - j * rp)] = v[u];
      }
    }
  }
}

// Streaming phase over rows [b0, b1): s = core S (row-dots) with S in LDS region s2,
// then v[n] = sum_b U^beta[n][b] s[b] (column axpy).  A whole item adds conj(v) to V
// (atomic adds); a row block of a split item (part_out != nullptr) stores v as its
// partial-sum block.
template <typename T, int NT>
__device__ __forceinline__ void dis_stream(const typename Tr<T>::c* __restrict__ fac, const TuckItem& it,
                                           const Lds<T>& L, unsigned char* smem, int nrhs, int r, int b0, int b1,
                                           typename Tr<T>::c* part_out, typename Tr<T>::c* __restrict__ V) {
  using C = typename Tr<T>::c;
  using P = typename Tr<T>::pack;
  constexpr int E = Tr<T>::E;
  C* S2 = reinterpret_cast<C*>(smem) + L.s1;
  C* s3 = S2 + L.s2;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int Q = it.rt * it.rp;
  // s[b] = sum_q core[b][q] S[q]
  wave_rowdots<T>(fac + it.off_core, it.ld_c, b0 + wave, b1, (NT / 64), reinterpret_cast<const P*>(S2),
                  round_up(Q, E) / E, s3, lane);
  __syncthreads();
  // V[n] += conj(sum_b U^beta[n][b] s[b])
  const int nb = it.nb;
  const int npk = round_up(nb, E) / E;
  C* Vo = V + it.row0 * nrhs + r;
  for (int base = 0; base < npk; base += NT * kColPacks) {
    P acc[kColPacks];
#pragma unroll
    for (int j = 0; j < kColPacks; ++j) acc[j] = pzero<P>();
    block_colaxpy<T, NT>(fac + it.off_ubt + (int64_t)b0 * it.ld_ub, it.ld_ub, b1 - b0, s3 + b0, npk, base, tid,
                         acc);
#pragma unroll
    for (int j = 0; j < kColPacks; ++j) {
      const int p = base + tid + NT * j;
      if (p < npk && part_out) {
        reinterpret_cast<P*>(part_out)[p] = acc[j];
      } else if (p < npk) {
        const C* vals = reinterpret_cast<const C*>(&acc[j]);
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int n = p * E + e;
          if (n < nb) atomic_add_c(Vo + (int64_t)n * nrhs, conjc(vals[e]));
        }
      }
    }
  }
}

// ---------------------------------------------------------------------- kernels

// Aggregation of one work unit: a whole item (stream, angular phase, F written) or a
// row block of a split item (its partial t stored for the finishing kernel).
template <typename T, int NT>
__device__ __forceinline__ void agg_unit(const typename Tr<T>::c* __restrict__ fac, const TuckWork& work,
                                         const TuckSplit* splits, const Lds<T>& L,
                                         unsigned char* smem, int n_theta, int n_phi, int nrhs, int r,
                                         const typename Tr<T>::c* __restrict__ x, typename Tr<T>::c* __restrict__ F,
                                         typename Tr<T>::c* part, int64_t part_stride) {
  using C = typename Tr<T>::c;
  const TuckItem& it = work.it;
  const TuckUnit& u = work.u;
  if (u.split < 0) {
    C* ts = reinterpret_cast<C*>(smem);  // t over x
    agg_stream<T, NT>(fac, it, L, smem, nrhs, r, x, 0, it.rb, ts);
    __syncthreads();
    agg_angular<T, NT>(it, global_angular<T>(fac, it), ts + L.r1, ts, n_theta, n_phi, nrhs, r, F);
  } else {
    const TuckSplit sp = splits[u.split];
    agg_stream<T, NT>(fac, it, L, smem, nrhs, r, x, u.b0, u.b1,
                      part + r * part_stride + sp.agg_off + (int64_t)u.sub * sp.q_pad);
  }
}

// Disaggregation of one work unit: angular phase, then the stream over the unit's
// rows; a whole item adds into V, a row block stores its partial v.
template <typename T, int NT>
__device__ __forceinline__ void dis_unit(const typename Tr<T>::c* __restrict__ fac, const TuckWork& work,
                                         const TuckSplit* splits, const Lds<T>& L,
                                         unsigned char* smem, int n_theta, int n_phi, int nrhs, int r,
                                         const typename Tr<T>::c* __restrict__ G, typename Tr<T>::c* __restrict__ V,
                                         typename Tr<T>::c* part, int64_t part_stride) {
  using C = typename Tr<T>::c;
  const TuckItem& it = work.it;
  const TuckUnit& u = work.u;
  C* dst = nullptr;
  if (u.split >= 0) {
    const TuckSplit sp = splits[u.split];
    dst = part + r * part_stride + sp.dis_off + (int64_t)u.sub * sp.nb_pad;
  }
  C* s1 = reinterpret_cast<C*>(smem);
  const C* Gi = G + ((int64_t)it.frow * n_theta * n_phi) * nrhs + r;
  dis_angular<T, NT>(
      it, global_angular<T>(fac, it), s1, n_theta, n_phi, [&](int q) { return conjc(Gi[(int64_t)q * nrhs]); }, s1 + L.s1);
  __syncthreads();
  dis_stream<T, NT>(fac, it, L, smem, nrhs, r, u.b0, u.b1, dst, V);
}

// The general kernel: a unit's aggregation (x given), its disaggregation (G given), or with
// both a workgroup for each, neighbours in the launch, so that the few long items whose time a
// layout waits for run both at once.  Workgroups go to the eight XCDs round-robin: every other
// group of four pairs is swapped, so that no XCD runs one stage only.  (100 groups of mean 909
// and one of 17000 basis functions, complex64, a pass: 719 us; 1356 with a launch a stage.)
template <typename T>
__global__ __launch_bounds__(kGenThreads) void tucker_general_kernel(
    const typename Tr<T>::c* __restrict__ fac, const TuckWork* __restrict__ work, const TuckSplit* __restrict__ splits,
    TuckMax mx, int n_theta, int n_phi, int nrhs, const typename Tr<T>::c* __restrict__ x,
    typename Tr<T>::c* __restrict__ F, const typename Tr<T>::c* __restrict__ G, typename Tr<T>::c* __restrict__ V,
    typename Tr<T>::c* part, int64_t part_stride) {
  extern __shared__ __align__(16) unsigned char smem[];
  const bool pass = x != nullptr && G != nullptr;
  const int i = blockIdx.x;
  const bool dis = pass ? ((i ^ (i >> 3)) & 1) != 0 : x == nullptr;
  const TuckWork w = work[pass ? i >> 1 : i];
  if (dis)
    dis_unit<T, kGenThreads>(fac, w, splits, Lds<T>(mx), smem, n_theta, n_phi, nrhs, blockIdx.y, G, V, part, part_stride);
  else
    agg_unit<T, kGenThreads>(fac, w, splits, Lds<T>(mx), smem, n_theta, n_phi, nrhs, blockIdx.y, x, F, part, part_stride);
}

// ------------------------------------------------------------ row-streaming kernels
//
// One sweep over the rows b of an item's factors serves both stages.  Row b of
// U^beta^T and row b of the core take part in
//   y[b] = U_b . x,   t += core_b y[b]        (aggregation)
//   s[b] = core_b . S,   v += U_b s[b]        (disaggregation)
// and every product above needs only row b, so a pass reads each factor once, not once
// per stage.  A row's packs (U_b first, then core_b) are cut into slices of 64; slice
// w + NW j belongs to wavefront w (NW wavefronts), whose lanes hold one pack each of
// the KR rows in work and of the KR rows being loaded, the matching packs of x or S and
// the running sums of v or t in registers.  Per KR rows the dot products are summed
// over the wavefront by a halving exchange (each step adds and halves the values a lane
// carries), over the wavefronts through LDS (one barrier), and return as wavefront-
// uniform scalars for the axpy.
//
// The sweep is bound by HBM.  A stage alone runs the same code with the other stage's
// vector zero (or its products left out), so a pass equals its two stages bit for bit.

// Sum of v and its partner lane across lane bit BIT (BIT = 4 pairs lanes i and 7 - i of
// eight, which later steps over bits 2 and 1 complete to the same sums).
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
template <int BIT>
__device__ __forceinline__ uint32_t partner(uint32_t v) {
  static_assert(BIT == 8 || BIT == 4 || BIT == 2 || BIT == 1, "within a row of 16 lanes");
  constexpr int ctrl = BIT == 8 ? 0x128 /* row_ror:8 */ : BIT == 4 ? 0x141 /* row_half_mirror */
                       : BIT == 2 ? 0x4E /* quad_perm 2,3,0,1 */ : 0xB1 /* quad_perm 1,0,3,2 */;
  return dpp_u32<ctrl>(v);
}
template <int BIT>
__device__ __forceinline__ float partner(float v) {
  return __uint_as_float(partner<BIT>(__float_as_uint(v)));
}
template <int BIT>
__device__ __forceinline__ double partner(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = partner<BIT>((uint32_t)u), hi = partner<BIT>((uint32_t)(u >> 32));
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
// The value of the lane 4 further on in the row of 16.
__device__ __forceinline__ float rotate4(float v) { return __uint_as_float(dpp_u32<0x124>(__float_as_uint(v))); }
__device__ __forceinline__ double rotate4(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = dpp_u32<0x124>((uint32_t)u), hi = dpp_u32<0x124>((uint32_t)(u >> 32));
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
// v_permlane32_swap (v_permlane16_swap) exchanges the upper half (odd rows of 16) of a
// with the lower half (even rows) of b.
template <int BIT>
__device__ __forceinline__ void lane_swap(uint32_t& a, uint32_t& b) {
  typedef unsigned int u2 __attribute__((ext_vector_type(2)));
  u2 r;
  if constexpr (BIT == 32)
    r = __builtin_bit_cast(u2, __builtin_amdgcn_permlane32_swap(a, b, false, false));
  else
    r = __builtin_bit_cast(u2, __builtin_amdgcn_permlane16_swap(a, b, false, false));
  a = r[0];
  b = r[1];
}
template <int BIT>
__device__ __forceinline__ float swap_add(float a, float b) {
  uint32_t x = __float_as_uint(a), y = __float_as_uint(b);
  lane_swap<BIT>(x, y);
  return __uint_as_float(x) + __uint_as_float(y);
}
template <int BIT>
__device__ __forceinline__ double swap_add(double a, double b) {
  const uint64_t u = (uint64_t)__double_as_longlong(a), w = (uint64_t)__double_as_longlong(b);
  uint32_t al = (uint32_t)u, ah = (uint32_t)(u >> 32), bl = (uint32_t)w, bh = (uint32_t)(w >> 32);
  lane_swap<BIT>(al, bl);
  lane_swap<BIT>(ah, bh);
  return __longlong_as_double((long long)(((uint64_t)ah << 32) | al)) +
         __longlong_as_double((long long)(((uint64_t)bh << 32) | bl));
}
// Lanes with bit BIT clear receive a's sum over the lane pair, lanes with it set b's.
template <int BIT, typename T>
__device__ __forceinline__ T fold2(T a, T b, int lane) {
  if constexpr (BIT >= 16) {
    return swap_add<BIT>(a, b);
  } else {
    const bool up = lane & BIT;
    const T keep = up ? b : a, send = up ? a : b;
    return keep + partner<BIT>(send);
  }
}
template <int BIT, typename T>
__device__ __forceinline__ T pair_add(T v) {
  if constexpr (BIT >= 16)
    return swap_add<BIT>(v, v);
  else
    return v + partner<BIT>(v);
}
// Sums of v[0 .. NV) (NV a power of two, at most 64) over the wavefront: lane l returns
// the total of value l / (64 / NV).
template <int NV, int BIT, typename T>
__device__ __forceinline__ T wave_fold(T (&v)[NV], int lane) {
  if constexpr (NV > 1) {
    T h[NV / 2];
#pragma unroll
    for (int i = 0; i < NV / 2; ++i) h[i] = fold2<BIT>(v[i], v[i + NV / 2], lane);
    return wave_fold<NV / 2, BIT / 2>(h, lane);
  } else if constexpr (BIT >= 1) {
    T h[1] = {pair_add<BIT>(v[0])};
    return wave_fold<1, BIT / 2>(h, lane);
  } else {
    return v[0];
  }
}
// Sum over the lanes that differ in the bits from FROM (4 or more) up to 32.  (In a row of
// 16, rotations by 4 and then by 8 reach the four lanes equal in bits 1 and 0.)
template <int FROM, typename T>
__device__ __forceinline__ T high_add(T v) {
  static_assert(FROM >= 4, "the rotation by 4 keeps bits 1 and 0");
  if constexpr (FROM == 4)
    return high_add<8>(v + rotate4(v));
  else if constexpr (FROM < 64)
    return high_add<FROM * 2>(pair_add<FROM>(v));
  else
    return v;
}
__device__ __forceinline__ float lane_value(float v, int lane) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), lane));
}
__device__ __forceinline__ double lane_value(double v, int lane) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// LDS of a row-streaming workgroup (complex elements; red in bytes):
//   vec    [RB][row]  x (padded to whole packs), then S of the disaggregation, later t
//   inter  the angular intermediate of either stage
//   gs     staged conj(G) of one right-hand side, us the staged angular factors (0 unstaged)
//   red    the wavefronts' partial dot products, double buffered
template <typename T>
struct StreamLds {
  int vecs, row, inter, gs, us, red;
  static constexpr int kRedValues = 16;  // dot products of a step per right-hand side, at most
  static constexpr int kTooLarge = 1 << 28;
  __host__ __device__ __forceinline__ StreamLds(const TuckMax& mx, int nw, int rb, bool staged, bool dis)
      : vecs(rb),
        row(round_up(mx.row, 2)),
        inter(round_up(mx.t3, 2)),
        gs(staged && dis ? round_up(mx.nt * mx.np, 2) : 0),
        us(staged ? staged_factors(mx) : 0),
        red(nw > 1 ? 2 * nw * kRedValues * rb * (int)sizeof(T) : 0) {}
  // (a grid of millions of angles times a rank passes an int; a size beyond any LDS stands for it)
  static __host__ __device__ __forceinline__ int staged_factors(const TuckMax& mx) {
    const int64_t n = (((int64_t)mx.nt * (mx.rt | 1) + 1) & ~1ll) + (((int64_t)mx.np * (mx.rp | 1) + 1) & ~1ll);
    return n < kTooLarge ? (int)n : kTooLarge;
  }
  __host__ __device__ size_t bytes() const {
    return ((size_t)vecs * row + inter + gs + us) * sizeof(typename Tr<T>::c) + red;
  }
};

// Rows per step, and steps whose rows are held (one in work, the others being loaded), for
// J slices per wavefront: 32 to 120 registers of row data a lane.  One right-hand side's short
// rows hold 2 steps, for the registers that a fifth wavefront needs.  A row of 5 slices and
// more keeps one workgroup on a CU, so its own loads must cover their latency: 3 steps, as
// long as nothing spills (with 2 steps, instances for 8, 10 and 16 slices only and the vector
// in LDS, one of which spilled, 140 items of mean 1.7M elements, complex64, 2911 us, now 797;
// and 200 of mean 260k, complex128, 386 us, now 278; one read a stage took 931 and 324 us).
constexpr int rows_per_step(int J) { return J == 1 ? 4 : (J == 2 ? 2 : 1); }
constexpr int steps_held(int J, int RB, bool f64) {
  if (J > 10 || (J == 4 && f64)) return 2;
  return J <= 2 && RB == 1 ? 2 : 3;
}

__device__ __forceinline__ float4 pkeep(float4 v, bool k) {
  return make_float4(k ? v.x : 0.f, k ? v.y : 0.f, k ? v.z : 0.f, k ? v.w : 0.f);
}
__device__ __forceinline__ double2 pkeep(double2 v, bool k) { return make_double2(k ? v.x : 0.0, k ? v.y : 0.0); }

// If `now`: d[0] takes the running sum d[1], which starts again from zero.
template <typename C>
__device__ __forceinline__ void restart(C (&d)[2], bool now) {
  d[0].x = now ? d[1].x : d[0].x;
  d[0].y = now ? d[1].y : d[0].y;
  d[1].x = now ? 0 : d[1].x;
  d[1].y = now ? 0 : d[1].y;
}

// The sweep over rows [b0, b1) with J slices per wavefront.  `ub` and `cb`: row 0 of
// U^beta^T and of the core (npu and npc packs per row); vec: the RB vectors in LDS, vrow packs apart.  On return acc[r][j] of lane l holds pack
// l of slice w + NW j of [v | t] for right-hand side r.
template <typename T, int NT, int J, int RB>
__device__ __forceinline__ void sweep_rows(const typename Tr<T>::pack* ub, const typename Tr<T>::pack* cb, int npu,
                                           int npc, int b0, int b1,
                                           const typename Tr<T>::pack* vec, int vrow, T* red, int wave, int lane,
                                           bool agg, bool dis, typename Tr<T>::pack (&acc)[RB][J]) {
  using C = typename Tr<T>::c;
  using P = typename Tr<T>::pack;
  constexpr int NW = NT / 64;
  constexpr int KR = rows_per_step(J), D = steps_held(J, RB, sizeof(T) == 8);
  constexpr int NV = 4 * KR * RB;
  constexpr bool kVecRegs = RB == 1;
  constexpr int kAux = NT >= 256 ? 2 : 0;  // non-temporal
  static_assert(NV <= 64 && NV <= StreamLds<T>::kRedValues * RB, "dot products per step");
  const int nsu = (npu + 63) >> 6, ns = nsu + ((npc + 63) >> 6);

  // slice j of this wavefront and this lane's pack in it; a slice beyond the row repeats the
  // wavefront's first one and, like a lane beyond the row, meets a zero vector.  All but
  // the lane offsets is wavefront-uniform and the step has no branch: buffer loads take
  // the item's base, a 32-bit lane offset and a scalar row offset, and the waits for them
  // count exactly.
  uint32_t ld[J], off[J];
  int voff[J];
  bool isu[J], live[J];
  const uint64_t at = (uint64_t)ub;
  const uint64_t at0 = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at) |
                       (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(at >> 32)) << 32;
  const auto rows = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(at0), 0, -1, 0x00027000);
  const uint32_t core = (uint32_t)((uint64_t)cb - at);
#pragma unroll
  for (int j = 0; j < J; ++j) {
    int s = wave + NW * j;
    const bool in = s < ns;
    s = in ? s : (wave < ns ? wave : 0);
    const bool u = s < nsu;
    isu[j] = in && u;
    const int p = 64 * (u ? s : s - nsu) + lane, np = u ? npu : npc;
    ld[j] = (uint32_t)np * sizeof(P);
    const int q = min(p, np - 1);
    off[j] = (uint32_t)q * sizeof(P) + (u ? 0u : core);
    live[j] = in && p < np;
    voff[j] = q + (u ? 0 : npu);
  }
  // first core slice of the wavefront: the sum over slices restarts there
  int jc = 0;
#pragma unroll
  for (int j = 0; j < J; ++j) jc += isu[j] ? 1 : 0;
  // A stage alone needs only the dot products with its vector and only its own sums.  Several
  // right-hand sides leave the absent stage's out, per wavefront (300 items of mean 58k elements,
  // complex64, 256 threads, the two stages with 3 and 5: 321 and 460 us, now 284 and 413); for one
  // the branches cost more than the products (4 wavelengths: both stages 1490 us, 1874 with them).
  const bool dots = RB == 1 || (agg && jc > 0) || (dis && jc < J);
  const bool sums = RB == 1 || (agg && jc < J) || (dis && jc > 0);
  P xv[kVecRegs ? J : 1];
  if constexpr (kVecRegs) {
#pragma unroll
    for (int j = 0; j < J; ++j) xv[j] = live[j] ? vec[voff[j]] : pzero<P>();
  }
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int j = 0; j < J; ++j) acc[r][j] = pzero<P>();

  auto load = [&](P (&u)[KR][J], int b) {
#pragma unroll
    for (int k = 0; k < KR; ++k) {
      const uint32_t row = (uint32_t)min(b + k, b1 - 1);  // (rows past the end are loaded, not used)
#pragma unroll
      for (int j = 0; j < J; ++j)
        u[k][j] = __builtin_bit_cast(P, __builtin_amdgcn_raw_buffer_load_b128(rows, off[j], row * ld[j], kAux));
    }
  };
  int par = 0;
  auto step = [&](const P (&u)[KR][J], int b) {
    T tot = T(0);
    if (dots) {
      C d[KR][RB][2];  // dot products of the row with x (U_b) and S (core_b)
#pragma unroll
      for (int k = 0; k < KR; ++k)
#pragma unroll
        for (int r = 0; r < RB; ++r) d[k][r][0] = d[k][r][1] = czero<C>();
#pragma unroll
      for (int j = 0; j < J; ++j) {
        P xr[RB];
#pragma unroll
        for (int r = 0; r < RB; ++r) {
          if constexpr (kVecRegs) {
            xr[r] = xv[j];
          } else {
            xr[r] = pkeep(vec[r * vrow + voff[j]], live[j]);
          }
        }
#pragma unroll
        for (int k = 0; k < KR; ++k)
#pragma unroll
          for (int r = 0; r < RB; ++r) {
            if (j > 0) restart(d[k][r], j == jc);  // U_b's sum up to slice jc, then core_b's
            pdot(d[k][r][1], u[k][j], xr[r]);
          }
      }
#pragma unroll
      for (int k = 0; k < KR; ++k)
#pragma unroll
        for (int r = 0; r < RB; ++r) restart(d[k][r], jc == J);
      T v[NV];
#pragma unroll
      for (int k = 0; k < KR; ++k)
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
          for (int m = 0; m < 2; ++m) {
            v[((k * RB + r) * 2 + m) * 2] = d[k][r][m].x;
            v[((k * RB + r) * 2 + m) * 2 + 1] = d[k][r][m].y;
          }
      tot = wave_fold<NV, 32>(v, lane);
    }
    constexpr int kSpan = 64 / NV;  // lanes per value
    int stride = kSpan;
    if constexpr (NW > 1) {
      T* rd = red + par * NW * NV;
      par ^= 1;
      if (lane % kSpan == 0) rd[wave * NV + lane / kSpan] = tot;
      __syncthreads();
      tot = T(0);
#pragma unroll
      for (int w0 = 0; w0 < NW; w0 += kSpan) {
        const int w = w0 + lane / NV;
        const T part = rd[min(w, NW - 1) * NV + lane % NV];
        tot += w < NW ? part : T(0);
      }
      tot = high_add<NV>(tot);
      stride = 1;
    }
    if (!sums) return;
#pragma unroll
    for (int k = 0; k < KR; ++k) {
      const bool in = b + k < b1;
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const int i = (k * RB + r) * 4;
        C y = {lane_value(tot, i * stride), lane_value(tot, (i + 1) * stride)};
        C sv = {lane_value(tot, (i + 2) * stride), lane_value(tot, (i + 3) * stride)};
        if (KR > 1) {
          y = {in ? y.x : 0, in ? y.y : 0};
          sv = {in ? sv.x : 0, in ? sv.y : 0};
        }
#pragma unroll
        for (int j = 0; j < J; ++j) {
          const C c = {j < jc ? sv.x : y.x, j < jc ? sv.y : y.y};
          paxpy(acc[r][j], u[k][j], c);
        }
      }
    }
  };
  P u[D][KR][J];
#pragma unroll
  for (int i = 0; i + 1 < D; ++i) {
    load(u[i], b0 + i * KR);
    __builtin_amdgcn_sched_barrier(0);  // in step order, so that the waits in the loop are exact
  }
  for (int b = b0; b < b1;) {
#pragma unroll
    for (int i = 0; i < D; ++i) {
      load(u[(i + D - 1) % D], b + (D - 1) * KR);
      step(u[i], b);
      b += KR;
      if (b >= b1) break;
    }
  }
}

template <typename T>
struct StreamArgs {
  const typename Tr<T>::c* fac;
  const TuckWork* work;
  const TuckSplit* splits;
  int n_units, n_theta, n_phi, nrhs, rstep, n_rblk;
  int blk_x;  // a stage's grid: blocks of a unit along x (1 or n_rblk; else along y)
  TuckMax mx;
  int staged;
  const typename Tr<T>::c* x;  // nullptr: no aggregation
  typename Tr<T>::c* F;
  const typename Tr<T>::c* G;  // nullptr: no disaggregation
  typename Tr<T>::c* V;
  typename Tr<T>::c* part;
  int64_t part_stride;
  int32_t* next;  // work counter of a persistent launch (nullptr: one workgroup per entry)
};

// The sweep and its outputs: t to LDS (`vec`'s S region; a split item's row block stores
// it as its partial sums), conj(v) added to V (or stored as partial sums).
template <typename T, int NT, int J, int RB>
__device__ __forceinline__ void sweep_unit(const StreamArgs<T>& a, const TuckItem& it, const TuckUnit& u, int r0,
                                           int nr, typename Tr<T>::c* vec, int vrow, T* red) {
  using C = typename Tr<T>::c;
  using P = typename Tr<T>::pack;
  constexpr int E = Tr<T>::E, NW = NT / 64;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int npu = it.ld_ub / E, npc = it.ld_c / E;
  const int nsu = (npu + 63) >> 6, ns = nsu + ((npc + 63) >> 6);
  const bool agg = a.x != nullptr, dis = a.G != nullptr;
  P acc[RB][J];
  sweep_rows<T, NT, J, RB>(reinterpret_cast<const P*>(a.fac + it.off_ubt),
                           reinterpret_cast<const P*>(a.fac + it.off_core), npu, npc, u.b0, u.b1,
                           reinterpret_cast<const P*>(vec), vrow / E, red, wave, lane, agg, dis, acc);
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int s = wave + NW * j;
    if (s >= ns) break;
    const bool isu = s < nsu;
    const int p = 64 * (isu ? s : s - nsu) + lane;
    if (p >= (isu ? npu : npc) || !(isu ? dis : agg)) continue;
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      if (r >= nr) break;
      if (u.split >= 0) {
        const TuckSplit sp = a.splits[u.split];
        const int64_t v_at = sp.dis_off + (int64_t)u.sub * sp.nb_pad, t_at = sp.agg_off + (int64_t)u.sub * sp.q_pad;
        C* dst = a.part + (r0 + r) * a.part_stride + (isu ? v_at : t_at);
        reinterpret_cast<P*>(dst)[p] = acc[r][j];
      } else if (!isu) {
        reinterpret_cast<P*>(vec + r * vrow + it.ld_ub)[p] = acc[r][j];
      } else {
        const C* vals = reinterpret_cast<const C*>(&acc[r][j]);
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int n = p * E + e;
          if (n < it.nb) atomic_add_c(a.V + (it.row0 + n) * a.nrhs + r0 + r, conjc(vals[e]));
        }
      }
    }
  }
}

// *p through the scalar cache, for a uniform p: what it points at is constant while kernels
// run.
__device__ __forceinline__ TuckWork const_load(const TuckWork* p) {
  struct Words {
    uint32_t w[sizeof(TuckWork) / 4];
  } v;
  typedef const uint32_t __attribute__((address_space(4))) * Const;
  const Const c = (Const)(uint64_t)p;
#pragma unroll
  for (unsigned i = 0; i < sizeof(TuckWork) / 4; ++i) v.w[i] = c[i];
  return __builtin_bit_cast(TuckWork, v);
}

// One work entry: unit iu and block blk of at most RB right-hand sides.  In a pass, and in a
// stage without split items, the entries of a unit follow each other, so that the second and
// later blocks find the factors in the memory-side cache.
template <typename T, int NT, int JMAX, int RB>
__device__ __forceinline__ void stream_entry(const StreamArgs<T>& a, const StreamLds<T>& L, unsigned char* smem,
                                             int iu, int blk, int32_t& next_entry) {
  using C = typename Tr<T>::c;
  constexpr int E = Tr<T>::E, NW = NT / 64;
  const int tid = threadIdx.x;
  // (the list is constant while kernels run: scalar loads)
  const TuckWork work = const_load(a.work + iu);
  const TuckUnit& u = work.u;
  const TuckItem& it = work.it;
  const int r0 = blk * a.rstep, nr = min(a.rstep, a.nrhs - r0);
  C* vec = reinterpret_cast<C*>(smem);
  C* inter = vec + RB * L.row;
  C* gs = inter + L.inter;
  C* us = gs + L.gs;
  T* red = reinterpret_cast<T*>(us + L.us);
  const bool staged = a.staged && !it.ident;
  const C* Gi = a.G ? a.G + ((int64_t)it.frow * a.n_theta * a.n_phi) * a.nrhs + r0 : nullptr;
  stage_in<T, NT>(a.fac, it, a.n_theta, a.n_phi, a.nrhs, a.x ? a.x + r0 : nullptr, nr, vec, L.row, Gi,
                  staged && a.G ? gs : nullptr, staged && (a.G || u.split < 0) ? us : nullptr);
  // zeros: x's padding to whole packs (all of it without an aggregation), absent columns
  for (int r = 0; r < RB; ++r) {
    C* v = vec + r * L.row;
    const bool col = r < nr;
    for (int n = (col && a.x ? it.nb : 0) + tid; n < it.ld_ub; n += NT) v[n] = czero<C>();
    if (!col || !a.G)
      for (int q = tid; q < it.ld_c; q += NT) v[it.ld_ub + q] = czero<C>();
  }
  __syncthreads();
  if (a.G) {
    for (int r = 0; r < nr; ++r) {
      C* S = vec + r * L.row + it.ld_ub;
      if (r > 0) {  // the previous column's products have read their operands
        __syncthreads();
        if (staged) {
          stage_in<T, NT>(a.fac, it, a.n_theta, a.n_phi, a.nrhs, nullptr, 1, nullptr, 0, Gi + r, gs, nullptr);
          __syncthreads();
        }
      }
      if (staged)
        dis_angular<T, NT>(
            it, staged_angular<T>(us, it, a.n_theta), inter, a.n_theta, a.n_phi, [&](int q) { return gs[q]; }, S);
      else
        dis_angular<T, NT>(
            it, global_angular<T>(a.fac, it), inter, a.n_theta, a.n_phi, [&](int q) { return conjc(Gi[(int64_t)q * a.nrhs + r]); }, S);
    }
    __syncthreads();
  }
  const int ns = ((it.ld_ub / E + 63) >> 6) + ((it.ld_c / E + 63) >> 6);
  const int j = (ns + NW - 1) / NW;
  if constexpr (JMAX == 2) {
    if (j <= 1)
      sweep_unit<T, NT, 1, RB>(a, it, u, r0, nr, vec, L.row, red);
    else
      sweep_unit<T, NT, 2, RB>(a, it, u, r0, nr, vec, L.row, red);
  } else if constexpr (JMAX == 4) {
    if (j <= 1)
      sweep_unit<T, NT, 1, RB>(a, it, u, r0, nr, vec, L.row, red);
    else if (j == 2)
      sweep_unit<T, NT, 2, RB>(a, it, u, r0, nr, vec, L.row, red);
    else if (j == 3)
      sweep_unit<T, NT, 3, RB>(a, it, u, r0, nr, vec, L.row, red);
    else
      sweep_unit<T, NT, 4, RB>(a, it, u, r0, nr, vec, L.row, red);
  } else {
    // (a slice more than the row has is loaded and not used)
    if (j <= 2)
      sweep_unit<T, NT, 2, RB>(a, it, u, r0, nr, vec, L.row, red);
    else if (j <= 4)
      sweep_unit<T, NT, 4, RB>(a, it, u, r0, nr, vec, L.row, red);
    else if (j == 5)
      sweep_unit<T, NT, 5, RB>(a, it, u, r0, nr, vec, L.row, red);
    else if (j == 6)
      sweep_unit<T, NT, 6, RB>(a, it, u, r0, nr, vec, L.row, red);
    else if (j == 7)
      sweep_unit<T, NT, 7, RB>(a, it, u, r0, nr, vec, L.row, red);
    else if (j == 8 || JMAX == 8)
      sweep_unit<T, NT, 8, RB>(a, it, u, r0, nr, vec, L.row, red);
    else if (j <= 10)
      sweep_unit<T, NT, 10, RB>(a, it, u, r0, nr, vec, L.row, red);
    else if (j == 11)
      sweep_unit<T, NT, 11, RB>(a, it, u, r0, nr, vec, L.row, red);
    else
      sweep_unit<T, NT, 12, RB>(a, it, u, r0, nr, vec, L.row, red);
  }
  if (a.next && tid == 0) next_entry = atomicAdd(a.next, 1);
  if (a.x == nullptr || u.split >= 0) return;
  for (int r = 0; r < nr; ++r) {
    __syncthreads();
    const C* ts = vec + r * L.row + it.ld_ub;
    if (staged)
      agg_angular<T, NT>(it, staged_angular<T>(us, it, a.n_theta), inter, ts, a.n_theta, a.n_phi, a.nrhs, r0 + r, a.F);
    else
      agg_angular<T, NT>(it, global_angular<T>(a.fac, it), inter, ts, a.n_theta, a.n_phi, a.nrhs, r0 + r, a.F);
  }
}

// A pass is persistent: as many workgroups as the CUs hold at once, each taking the next
// entry of the longest-first list from the work counter, which the V-zeroing kernel
// before it sets to zero (with one workgroup per entry the hardware refilled a CU's free
// slot only tens of microseconds after a unit of a small-box layout ended).  A stage
// alone runs one workgroup per entry.
template <typename T, int NT, int JMAX, int RB>
__global__ __launch_bounds__(NT)
__attribute__((amdgpu_waves_per_eu(RB > 1 || JMAX > 4 ? 2 : (JMAX == 2 ? 5 : 4))))
void tucker_pass_kernel(StreamArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int32_t take;  // (kPassStaticLds)
  const StreamLds<T> L(a.mx, NT / 64, RB, a.staged, a.G != nullptr);
  const int total = a.n_units * a.n_rblk;
  if (a.next == nullptr) {
    int32_t none;
    const int iu = blockIdx.x / a.blk_x;
    stream_entry<T, NT, JMAX, RB>(a, L, smem, iu, blockIdx.y + blockIdx.x - iu * a.blk_x, none);
    return;
  }
  int32_t mine = 0;  // (first thread) the next entry, taken when the current one's sweep is done
  if (threadIdx.x == 0) mine = atomicAdd(a.next, 1);
  for (;;) {
    if (threadIdx.x == 0) take = mine;
    __syncthreads();
    const int i = __builtin_amdgcn_readfirstlane(take);
    if (i >= total) break;  // uniform: every wavefront leaves
    const int iu = i / a.n_rblk;
    stream_entry<T, NT, JMAX, RB>(a, L, smem, iu, i - iu * a.n_rblk, mine);
    __syncthreads();  // the entry's last LDS reads and `take` are done before the next one
  }
}

// Finishing kernel of the split items, after the units: blocks [0, n_agg) sum the
// partial t of split entry blockIdx.x (in block order, so the result does not depend
// on the schedule) and run the angular phase into F; blocks [n_agg, gridDim.x) sum
// the partial v of split entry blockIdx.x - n_agg and add conj(v) to V.
constexpr int kFinishThreads = 512;
template <typename T>
struct FinishLds {
  int q, inter, stage;
  __host__ __device__ __forceinline__ FinishLds(const TuckMax& mx, bool staged)
      : q(round_up(round_up(mx.q, Tr<T>::E), 2)),
        inter(round_up(mx.t3, 2)),
        stage(staged ? StreamLds<T>::staged_factors(mx) : 0) {}
  __host__ __device__ size_t bytes() const { return ((size_t)q + inter + stage) * sizeof(typename Tr<T>::c); }
};
template <typename T>
__global__ __launch_bounds__(kFinishThreads) void tucker_finish_kernel(
    const typename Tr<T>::c* __restrict__ fac, const TuckItem* __restrict__ items,
    const TuckSplit* __restrict__ splits, int n_agg, TuckMax mx, int staged, int n_theta, int n_phi, int nrhs,
    const typename Tr<T>::c* __restrict__ part, int64_t part_stride, typename Tr<T>::c* __restrict__ F,
    typename Tr<T>::c* __restrict__ V) {
  using C = typename Tr<T>::c;
  constexpr int E = Tr<T>::E;
  extern __shared__ __align__(16) unsigned char smem[];
  const int r = blockIdx.y, tid = threadIdx.x;
  const bool agg = (int)blockIdx.x < n_agg;
  const TuckSplit sp = splits[agg ? blockIdx.x : blockIdx.x - n_agg];
  const TuckItem it = items[sp.item];
  const C* base = part + r * part_stride;
  if (agg) {
    const FinishLds<T> L(mx, staged);
    const int Q = it.rt * it.rp;
    C* ts = reinterpret_cast<C*>(smem);
    if (L.stage && !it.ident)
      stage_in<T, kFinishThreads>(fac, it, n_theta, n_phi, nrhs, nullptr, 1, nullptr, 0, nullptr, nullptr,
                                  ts + L.q + L.inter);
    for (int q = tid; q < round_up(Q, E); q += kFinishThreads) {
      C acc = czero<C>();
      if (q < Q)
        for (int s = 0; s < sp.n_parts; ++s) {
          const C v = base[sp.agg_off + (int64_t)s * sp.q_pad + q];
          acc.x += v.x;
          acc.y += v.y;
        }
      ts[q] = acc;
    }
    __syncthreads();
    C* inter = ts + L.q;
    if (L.stage && !it.ident)
      agg_angular<T, kFinishThreads>(it, staged_angular<T>(inter + L.inter, it, n_theta), inter, ts, n_theta, n_phi, nrhs, r, F);
    else
      agg_angular<T, kFinishThreads>(it, global_angular<T>(fac, it), inter, ts, n_theta, n_phi, nrhs, r, F);
  } else {
    C* Vo = V + it.row0 * nrhs + r;
    for (int n = tid; n < it.nb; n += kFinishThreads) {
      C acc = czero<C>();
      for (int s = 0; s < sp.n_parts; ++s) {
        const C v = base[sp.dis_off + (int64_t)s * sp.nb_pad + n];
        acc.x += v.x;
        acc.y += v.y;
      }
      atomic_add_c(Vo + (int64_t)n * nrhs, conjc(acc));
    }
  }
}

// v[0 .. n) = 0; with `counter`, also the pass kernel's work counter.
template <typename C>
__global__ __launch_bounds__(256) void zero_kernel(C* __restrict__ v, int64_t n, int32_t* __restrict__ counter) {
  if (counter && blockIdx.x == 0 && threadIdx.x == 0) *counter = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) v[i] = czero<C>();
}

template <typename C>
hipError_t zero(C* v, int64_t n, hipStream_t s, int32_t* counter = nullptr) {
  if (n <= 0 && !counter) return hipSuccess;
  const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 4096));
  hipLaunchKernelGGL(zero_kernel<C>, dim3((unsigned)blocks), dim3(256), 0, s, v, n, counter);
  return hipGetLastError();
}

// Grid of a persistent launch: the workgroups of `kernel` the CUs hold at once (by
// its registers and LDS), at most one per work entry.
template <typename K>
hipError_t persistent_grid(K kernel, int threads, size_t lds, int64_t entries, unsigned* blocks) {
  int dev = 0, n_cu = 0, per_cu = 0;
  hipError_t e;
  if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
  if ((e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
  if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(kernel), threads,
                                                        lds)) != hipSuccess)
    return e;
  *blocks = (unsigned)std::max<int64_t>(1, std::min<int64_t>(entries, (int64_t)std::max(per_cu, 1) * n_cu));
  return hipSuccess;
}

// One row per blockIdx.x, the row's elements split over blockIdx.y.
template <typename C>
__global__ __launch_bounds__(256) void zero_rows_kernel(C* __restrict__ base, const int32_t* __restrict__ rows,
                                                        int64_t row_elems) {
  C* row = base + (int64_t)rows[blockIdx.x] * row_elems;
  for (int64_t i = (int64_t)blockIdx.y * 256 + threadIdx.x; i < row_elems; i += (int64_t)gridDim.y * 256)
    row[i] = czero<C>();
}

}  // namespace

#ifndef TUCKFMM_STREAM_F64
hipError_t launch_zero_rows(size_t elem_bytes, void* base, const int32_t* rows, int n_rows, int64_t row_elems,
                            hipStream_t s) {
  if (n_rows <= 0 || row_elems <= 0) return hipSuccess;
  const unsigned ny = (unsigned)std::min<int64_t>(std::max<int64_t>(1, (row_elems + 2047) / 2048), 1024);
  if (elem_bytes == 16)
    hipLaunchKernelGGL(zero_rows_kernel<Tr<double>::c>, dim3((unsigned)n_rows, ny), dim3(256), 0, s,
                       static_cast<Tr<double>::c*>(base), rows, row_elems);
  else if (elem_bytes == 8)
    hipLaunchKernelGGL(zero_rows_kernel<Tr<float>::c>, dim3((unsigned)n_rows, ny), dim3(256), 0, s,
                       static_cast<Tr<float>::c*>(base), rows, row_elems);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}
#endif

// Kernel of a fit (see stream_fits).
#define TFMM_STREAM_CASE(nt, jm, r)                            \
  if (f.threads == nt && f.jmax == jm && f.rb == r) {          \
    constexpr int NT = nt, JMAX = jm, RB = r;                  \
    return launch_stream_kernel<T, NT, JMAX, RB>(a, f, entries, s); \
  }

// The general kernel's LDS.
template <typename T>
size_t tucker_lds_bytes(const TuckMax& mx) {
  return Lds<T>(mx).bytes();
}

// Whether work entries of rb right-hand sides each, in workgroups of `threads`, still hold a
// workgroup of 512 threads per CU.  Below that (layouts of few units) sharing a read of the
// factors leaves CUs idle, and every right-hand side is an entry of its own: 100 groups of 2
// wavelengths, complex64, 2 right-hand sides, a pass and the two stages, 169 and 368 us, shared
// 237 and 415; 8 groups of 240 basis functions 33 and 50, shared 48 and 53; with 3 of them the
// 100 groups have enough entries: 205 and 475, shared 241 and 427.
constexpr int64_t kFillThreads = 256 * 512;
static bool entries_fill(int n_units, int nrhs, int rb, int threads) {
  return (int64_t)n_units * ((nrhs + rb - 1) / rb) * threads >= kFillThreads;
}

static int slices_per_wave(const TuckMax& mx, int threads) { return (mx.slices + threads / 64 - 1) / (threads / 64); }

// The row-streaming kernel for workgroups of `threads` (more where the longest row needs
// them) and nrhs right-hand sides; false if a row is too long for it or its LDS beyond
// mx.lds (the general kernel runs the layout then).  A wavefront's lanes hold up to 4
// slices of 64 packs in the kernels of 128 registers; longer rows take 8 or, with 512
// threads, 12 (more spill).  Two right-hand sides share a read of the factors where the row
// allows 4 slices and the entries fill the chip.  Four lose to two (1.5 wavelengths, 160
// groups, complex64, 5 right-hand sides, a pass and the stages: 289 and 534 us with two, 397 and
// 543 with four), but for 3 or a multiple of 4 where at least 256 threads hold at most 3 slices
// and twice the entries are left (3 right-hand sides: 1 wavelength, 300 groups, complex128, 394
// and 667 with two, 371 and 609 with four; 2 wavelengths, complex64, 256 groups 596 and 1040,
// 558 and 991; 100 groups 241 and 427, 394 and 700).  The angular operands are staged in LDS while a CU
// still holds kStageMinWaves wavefronts.
//
// Small complex64 items are bound by the latency of each unit's phases, which more workgroups
// on a CU hide.  With at most 2 slices the kernel fits 96 registers, so 5 wavefronts a SIMD
// (4000 items of mean 15k: 135 us with 4, 126 with 5; 6 spill, 134).  With 512
// threads 5 a SIMD hold no more workgroups than 4; in complex128 it was not tried.
template <typename T>
bool stream_fits(const TuckMax& mx, int n_units, int threads, int nrhs, bool dis, StreamFit* out) {
  for (; threads <= 512; threads *= 2) {
    const int nw = threads / 64, j = slices_per_wave(mx, threads);
    const bool small = j <= 2 && nrhs == 1 && threads <= 256 && sizeof(T) == 4;
    const int jmax = small ? 2 : (j <= 4 ? 4 : (j <= 8 ? 8 : (j <= 12 && threads == 512 ? 12 : 0)));
    if (!jmax) continue;
    int most = 1;
    if (jmax == 4 && nrhs > 1 && entries_fill(n_units, nrhs, 2, threads))
      most = threads >= 256 && j <= 3 && (nrhs + 1) % 4 < 2 && entries_fill(n_units, nrhs, 4, threads / 2) ? 4 : 2;
    for (int rb = most; rb >= 1; rb /= 2) {
      const size_t staged = StreamLds<T>(mx, nw, rb, true, dis).bytes();
      const size_t plain = StreamLds<T>(mx, nw, rb, false, dis).bytes();
      if (plain + kPassStaticLds > (size_t)mx.lds) continue;
      out->threads = threads;
      out->jmax = jmax;
      out->rb = rb;
      out->staged = mx.stage && staged + kPassStaticLds <= (size_t)mx.lds &&
                    (int)(kCuLds / (staged + kPassStaticLds)) * nw >= kStageMinWaves;
      out->lds = out->staged ? staged : plain;
      return true;
    }
  }
  return false;
}

#ifndef TUCKFMM_STREAM_F64
// The smallest workgroups of at least 128 threads whose wavefronts hold the longest row in 4
// slices, so that right-hand sides share reads and many units are in flight (160 groups of 1.5
// wavelengths, complex64, 5 right-hand sides, a pass and the stages: 289 and 534 us with 256
// threads, 373 and 595 with 512; with 128, which hold 7 slices and share nothing, 349 and 573).
// Two right-hand sides are one read either way and prefer 3 slices (1.5 wavelengths: 137 and 233
// with 512 threads, 181 and 323 with 256, 4 slices; 1 wavelength, 1000 groups: 269 and 421 with
// 256, 424 and 533 with 512).  Where the entries don't fill the chip, up to the size for one.
int multi_threads(const TuckMax& mx, int n_units, int threads, int nrhs) {
  const int most = nrhs == 2 ? 3 : 4;
  int t = 128;
  while (t < 512 && slices_per_wave(mx, t) > most) t *= 2;
  if (slices_per_wave(mx, t) > 4) return threads;
  for (; t <= 512; t *= 2) {
    if (entries_fill(n_units, nrhs, 2, t)) return t;
    if (t >= threads) break;
  }
  return threads;
}
#endif

template <typename T, int NT, int JMAX, int RB>
hipError_t launch_stream_kernel(StreamArgs<T> a, const StreamFit& f, int64_t entries, hipStream_t s) {
  // A stage: the column blocks of a unit follow each other (see stream_entry; 140 items of mean
  // 1.7M elements, complex64, the two stages with 3 right-hand sides: 2420 us in the other order,
  // now 2180).  Split items go by columns first: their units are alike, and 20 groups of 2
  // wavelengths took 5% less so.
  const bool flat = a.splits == nullptr && entries <= (1 << 22);
  a.blk_x = flat ? a.n_rblk : 1;
  dim3 grid((unsigned)(flat ? entries : a.n_units), (unsigned)(flat ? 1 : a.n_rblk));
  if (a.next) {
    const hipError_t e = persistent_grid(&tucker_pass_kernel<T, NT, JMAX, RB>, NT, f.lds, entries, &grid.x);
    if (e != hipSuccess) return e;
    grid.y = 1;
  }
  hipLaunchKernelGGL((tucker_pass_kernel<T, NT, JMAX, RB>), grid, dim3(NT), f.lds, s, a);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_stream(StreamArgs<T> a, const StreamFit& f, hipStream_t s) {
  const int64_t entries = (int64_t)a.n_units * a.n_rblk;
  // the counter runs past the entries by one per workgroup
  if (entries > INT32_MAX / 2) a.next = nullptr;
  if constexpr (sizeof(T) == 4) {
    TFMM_STREAM_CASE(64, 2, 1)
    TFMM_STREAM_CASE(128, 2, 1)
    TFMM_STREAM_CASE(256, 2, 1)
  }
  TFMM_STREAM_CASE(64, 4, 1)
  TFMM_STREAM_CASE(64, 4, 2)
  TFMM_STREAM_CASE(64, 8, 1)
  TFMM_STREAM_CASE(128, 4, 1)
  TFMM_STREAM_CASE(128, 4, 2)
  TFMM_STREAM_CASE(128, 8, 1)
  TFMM_STREAM_CASE(256, 4, 1)
  TFMM_STREAM_CASE(256, 4, 2)
  TFMM_STREAM_CASE(256, 4, 4)
  TFMM_STREAM_CASE(256, 8, 1)
  TFMM_STREAM_CASE(512, 4, 1)
  TFMM_STREAM_CASE(512, 4, 2)
  TFMM_STREAM_CASE(512, 4, 4)
  TFMM_STREAM_CASE(512, 8, 1)
  TFMM_STREAM_CASE(512, 12, 1)
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_finish(const TuckPlan& pl, int n_agg, int n_dis, int n_theta, int n_phi, int nrhs, void* F, void* V,
                         hipStream_t s) {
  using C = typename Tr<T>::c;
  if (n_agg + n_dis == 0) return hipSuccess;
  const bool staged = pl.mx.stage && FinishLds<T>(pl.mx, true).bytes() <= (size_t)pl.mx.lds;
  const size_t lds = n_agg ? FinishLds<T>(pl.mx, staged).bytes() : 0;
  // n_dis > 0 with n_agg == 0 runs the disaggregation blocks only: splits from 0
  hipLaunchKernelGGL(tucker_finish_kernel<T>, dim3(n_agg + n_dis, nrhs), dim3(kFinishThreads), lds, s,
                     static_cast<const C*>(pl.factors), pl.items, pl.splits, n_agg, pl.mx, staged ? 1 : 0, n_theta,
                     n_phi, nrhs, static_cast<const C*>(pl.part), pl.part_stride, static_cast<C*>(F),
                     static_cast<C*>(V));
  return hipGetLastError();
}

// Either stage (x or G nullptr) or both.
template <typename T>
hipError_t launch_units(const TuckPlan& pl, int threads, int n_theta, int n_phi, int nrhs, const void* x, void* F,
                        const void* G, void* V, bool persistent, hipStream_t s) {
  using C = typename Tr<T>::c;
  if (threads != 64 && threads != 128 && threads != 256 && threads != 512) return hipErrorInvalidValue;
  if (pl.n_splits > 0 && pl.part == nullptr) return hipErrorInvalidValue;
  if (persistent && pl.next == nullptr) return hipErrorInvalidValue;
  hipError_t e = hipSuccess;
  if (V && (e = zero(static_cast<C*>(V), pl.n_basis * nrhs, s, persistent ? pl.next : nullptr)) != hipSuccess) return e;
  if (pl.n_units == 0) return hipSuccess;
  StreamFit f;
  // a layout that fits one of the calls in full takes it in all of them, so that a pass
  // equals its stages
  if (stream_fits<T>(pl.mx, pl.n_units, threads, nrhs, true, &f)) {
    if (!G) stream_fits<T>(pl.mx, pl.n_units, threads, nrhs, false, &f);
    StreamArgs<T> a;
    a.fac = static_cast<const C*>(pl.factors);
    a.work = pl.work;
    a.splits = pl.splits;
    a.n_units = pl.n_units;
    a.n_theta = n_theta;
    a.n_phi = n_phi;
    a.nrhs = nrhs;
    a.n_rblk = (nrhs + f.rb - 1) / f.rb;
    a.rstep = (nrhs + a.n_rblk - 1) / a.n_rblk;
    a.mx = pl.mx;
    a.staged = f.staged;
    a.x = static_cast<const C*>(x);
    a.F = static_cast<C*>(F);
    a.G = static_cast<const C*>(G);
    a.V = static_cast<C*>(V);
    a.part = static_cast<C*>(pl.part);
    a.part_stride = pl.part_stride;
    a.next = persistent ? pl.next : nullptr;
    e = launch_stream<T>(a, f, s);
  } else {
    const Lds<T> L(pl.mx);
    hipLaunchKernelGGL((tucker_general_kernel<T>), dim3((unsigned)pl.n_units * (x && G ? 2 : 1), nrhs),
                       dim3(kGenThreads), x && G ? L.bytes() : (x ? L.agg_bytes() : L.dis_bytes()), s,
                       static_cast<const C*>(pl.factors), pl.work, pl.splits, pl.mx, n_theta, n_phi, nrhs,
                       static_cast<const C*>(x), static_cast<C*>(F), static_cast<const C*>(G), static_cast<C*>(V),
                       static_cast<C*>(pl.part), pl.part_stride);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return e;
  return launch_finish<T>(pl, x ? pl.n_splits : 0, G ? pl.n_splits : 0, n_theta, n_phi, nrhs, F, V, s);
}

template <typename T>
hipError_t launch_tucker_agg(const TuckPlan& pl, int threads, int n_theta, int n_phi, int nrhs, const void* x,
                             void* F, hipStream_t s) {
  return launch_units<T>(pl, threads, n_theta, n_phi, nrhs, x, F, nullptr, nullptr, false, s);
}

template <typename T>
hipError_t launch_tucker_disagg(const TuckPlan& pl, int threads, int n_theta, int n_phi, int nrhs, const void* G,
                                void* V, hipStream_t s) {
  return launch_units<T>(pl, threads, n_theta, n_phi, nrhs, nullptr, nullptr, G, V, false, s);
}

template <typename T>
hipError_t launch_tucker_pass(const TuckPlan& pl, int threads, int n_theta, int n_phi, int nrhs, const void* x,
                              void* F, const void* G, void* V, hipStream_t s) {
  return launch_units<T>(pl, threads, n_theta, n_phi, nrhs, x, F, G, V, true, s);
}

template size_t tucker_lds_bytes<Real>(const TuckMax&);
template bool stream_fits<Real>(const TuckMax&, int, int, int, bool, StreamFit*);
template hipError_t launch_tucker_agg<Real>(const TuckPlan&, int, int, int, int, const void*, void*, hipStream_t);
template hipError_t launch_tucker_disagg<Real>(const TuckPlan&, int, int, int, int, const void*, void*, hipStream_t);
template hipError_t launch_tucker_pass<Real>(const TuckPlan&, int, int, int, int, const void*, void*, const void*,
                                             void*, hipStream_t);

}  // namespace tuckfmm
