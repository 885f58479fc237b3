// Exact coarse solve u_0 = A_0^+ f_0 (P = 1) by global fast diagonalisation, FP64:
// one pass per direction with S_d^T, division by the sums of the eigenvalues, one pass
// per direction with S_d.  Three forms, with the same bits (coarse_form picks one):
//   one block   the whole vector and the matrices in LDS, every pass in one launch (bound
//               by LDS latency: 13 us for 2D 16 x 16, 1024 unknowns with a periodic mean,
//               before 13 launches of 3 to 5 us; 15.6 us for 7 x 5 x 6 elements, as passes
//               six launches)
//   planes      3D grids whose planes of directions 0 and 1 fit: forward along 0 and
//               1 per plane, forward, scaled and back along 2 per group of columns, back
//               along 1 and 0 per plane (three launches)
//   passes      the rest: one launch per direction and way (in dgmg.hip)
// Inside, values are in lexicographic order (direction 0 fastest) of the G_d nodes per
// direction (elements of two nodes, or the continuous lattice).
#pragma once

#include "kernels.hpp"

namespace dgmg {

struct CoarseDev {
  int dim = 3;
  int se = 0;                   // 1: continuous lattice vector (nl[d] nodes per direction)
  int nl[3] = {1, 1, 1};
  int N[3] = {1, 1, 1};
  const double* S[3] = {nullptr, nullptr, nullptr};    // G_d x G_d row-major
  const double* lam[3] = {nullptr, nullptr, nullptr};  // G_d
};
// Nodes of direction d.
__host__ __device__ inline int coarse_nodes(const CoarseDev& C, int d) {
  return d >= C.dim ? 1 : (C.se ? C.nl[d] : 2 * C.N[d]);
}
// Row pitch of a matrix in LDS: odd, so that columns spread over the banks.
__host__ __device__ inline int coarse_pitch(int G) { return G | 1; }
// Offset in the coarse vector of the node (i0, i1, i2).
__device__ __forceinline__ int64_t coarse_offset(const CoarseDev& C, int i0, int i1, int i2) {
  if (C.se) return i0 + (int64_t)C.nl[0] * (i1 + (int64_t)C.nl[1] * i2);
  const int64_t e = (i0 >> 1) + (int64_t)C.N[0] * ((i1 >> 1) + (int64_t)C.N[1] * (i2 >> 1));
  return C.dim == 3 ? e * 8 + ((i2 & 1) * 2 + (i1 & 1)) * 2 + (i0 & 1) : e * 4 + (i1 & 1) * 2 + (i0 & 1);
}

template <class T>
struct CoarseArgs {
  CoarseDev C;
  const T* f = nullptr;
  T* u = nullptr;
  const int* active = nullptr;
  int mean = 0;  // periodic in every direction: f less its mean, the mean-free solution
};

constexpr int COARSE_THREADS = 1024;
constexpr size_t COARSE_LDS = 150 * 1024;
// LDS of the one-block form: two vectors, the matrices, the eigenvalues.
inline size_t coarse_block_shmem(const CoarseDev& C) {
  size_t n = 1, m = 0;
  for (int d = 0; d < C.dim; ++d) {
    const size_t G = coarse_nodes(C, d);
    n *= G;
    m += G * (coarse_pitch((int)G) + 1);
  }
  return (2 * n + m) * sizeof(double);
}

__device__ __forceinline__ void coarse_matrix(const double* __restrict__ src, double* dst, int G) {
  const int p = coarse_pitch(G);
  for (int q = threadIdx.x; q < G * G; q += blockDim.x) dst[q / G * p + q % G] = src[q];
}

// out[.., I, ..] = sum_K M(K, I) in[.., K, ..] along a direction of G nodes with stride st,
// M(K, I) = S[K][I] (FWD) or S[I][K]; two lines per thread where there are that many, so
// that one matrix value serves both.  post maps (index, value).
template <bool FWD, class Post>
__device__ __forceinline__ void coarse_pass(const double* __restrict__ S, int G, int st, const double* in,
                                            double* out, int n, Post post) {
  const int nl = n / G, nh = (nl + 1) / 2, p = coarse_pitch(G);  // lines, of which nh first
  for (int q = threadIdx.x; q < nh * G; q += blockDim.x) {
    // node I of line l and of line l + nh; neighbouring threads on neighbouring values
    const int l = st == 1 ? q / G : q % nh, I = st == 1 ? q - l * G : q / nh;
    const int l1 = l + nh < nl ? l + nh : l;
    const int b0 = (l / st) * (G * st) + l % st, b1 = (l1 / st) * (G * st) + l1 % st;
    double s0 = 0.0, s1 = 0.0;
#pragma unroll 4
    for (int K = 0; K < G; ++K) {
      const double m = FWD ? S[K * p + I] : S[I * p + K];
      s0 = fma(m, in[b0 + K * st], s0);
      s1 = fma(m, in[b1 + K * st], s1);
    }
    out[b0 + I * st] = post(b0 + I * st, s0);
    if (l1 != l) out[b1 + I * st] = post(b1 + I * st, s1);
  }
}

// BATCH: one block per grid, its arguments in the work list.
template <class T, bool BATCH = false>
__global__ void __launch_bounds__(COARSE_THREADS) coarse_block_kernel(CoarseArgs<T> a0, BatchList<CoarseArgs<T>> bl) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ __align__(16) int sargs_raw[BATCH ? sizeof(CoarseArgs<T>) / sizeof(int) : 1];
  __shared__ double red[COARSE_THREADS / 64], mean;
  const CoarseArgs<T>* ap = &a0;
  if constexpr (BATCH) {
    CoarseArgs<T>* sargs = reinterpret_cast<CoarseArgs<T>*>(sargs_raw);
    const int* src = reinterpret_cast<const int*>(bl.descs + blockIdx.x);
    for (int i = threadIdx.x; i < (int)(sizeof(CoarseArgs<T>) / sizeof(int)); i += blockDim.x) sargs_raw[i] = src[i];
    __syncthreads();
    ap = sargs;
  }
  const CoarseDev& C = ap->C;
  if (inactive(ap->active)) return;
  const int G0 = coarse_nodes(C, 0), G1 = coarse_nodes(C, 1), G2 = coarse_nodes(C, 2), dim = C.dim;
  const int n = G0 * G1 * G2, tid = threadIdx.x, nth = blockDim.x;
  double* a = reinterpret_cast<double*>(smem_raw);
  double* b = a + n;
  double* S0 = b + n;
  double* S1 = S0 + G0 * coarse_pitch(G0);
  double* S2 = S1 + G1 * coarse_pitch(G1);
  double* l0 = S2 + (dim == 3 ? G2 * coarse_pitch(G2) : 0);
  double* l1 = l0 + G0;
  double* l2 = l1 + G1;
  coarse_matrix(C.S[0], S0, G0);
  coarse_matrix(C.S[1], S1, G1);
  for (int q = tid; q < G0; q += nth) l0[q] = C.lam[0][q];
  for (int q = tid; q < G1; q += nth) l1[q] = C.lam[1][q];
  if (dim == 3) {
    coarse_matrix(C.S[2], S2, G2);
    for (int q = tid; q < G2; q += nth) l2[q] = C.lam[2][q];
  }
  double s = 0.0;
  for (int q = tid; q < n; q += nth) {
    const int i0 = q % G0, r = q / G0;
    const double v = (double)ap->f[coarse_offset(C, i0, r % G1, r / G1)];
    a[q] = v;
    s += v;
  }
  const auto less_mean = [&](double* v, double sum) {  // v -= its mean (its values are the thread's own)
    sum = block_sum(sum, red);
    if (tid == 0) mean = sum / (double)n;
    __syncthreads();
    for (int q = tid; q < n; q += nth) v[q] -= mean;
  };
  if (ap->mean) less_mean(a, s);
  __syncthreads();
  const auto same = [](int, double v) { return v; };
  const auto scale = [&](int q, double v) {
    const int i0 = q % G0, r = q / G0;
    double den = l0[i0] + l1[r % G1];
    if (dim == 3) den += l2[r / G1];
    return den != 0.0 ? v / den : 0.0;
  };
  coarse_pass<true>(S0, G0, 1, a, b, n, same);
  __syncthreads();
  if (dim == 3) {
    coarse_pass<true>(S1, G1, G0, b, a, n, same);
    __syncthreads();
    coarse_pass<true>(S2, G2, G0 * G1, a, b, n, scale);
    __syncthreads();
    coarse_pass<false>(S2, G2, G0 * G1, b, a, n, same);
    __syncthreads();
    coarse_pass<false>(S1, G1, G0, a, b, n, same);
  } else {
    coarse_pass<true>(S1, G1, G0, b, a, n, scale);
    __syncthreads();
    coarse_pass<false>(S1, G1, G0, a, b, n, same);
  }
  __syncthreads();
  coarse_pass<false>(S0, G0, 1, b, a, n, same);
  __syncthreads();
  if (ap->mean) {
    s = 0.0;
    for (int q = tid; q < n; q += nth) s += a[q];
    less_mean(a, s);
  }
  for (int q = tid; q < n; q += nth) {  // each thread reads back what it wrote last (mean) or what the barrier made visible
    const int i0 = q % G0, r = q / G0;
    ap->u[coarse_offset(C, i0, r % G1, r / G1)] = (T)a[q];
  }
}

// Planes of directions 0 and 1 (one block each): forward from the coarse vector f into
// the lexicographic buffer w, or back from w into the coarse vector u.
template <class T, bool FWD>
__global__ void __launch_bounds__(256) coarse_planes_kernel(CoarseDev C, const T* __restrict__ f,
                                                            double* __restrict__ w, T* __restrict__ u,
                                                            const int* active) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  if (inactive(active)) return;
  const int G0 = coarse_nodes(C, 0), G1 = coarse_nodes(C, 1), n = G0 * G1, z = blockIdx.x;
  const int tid = threadIdx.x, nth = blockDim.x;
  double* a = reinterpret_cast<double*>(smem_raw);
  double* b = a + n;
  double* S0 = b + n;
  double* S1 = S0 + G0 * coarse_pitch(G0);
  coarse_matrix(C.S[0], S0, G0);
  coarse_matrix(C.S[1], S1, G1);
  for (int q = tid; q < n; q += nth)
    a[q] = FWD ? (double)f[coarse_offset(C, q % G0, q / G0, z)] : w[(int64_t)z * n + q];
  __syncthreads();
  const auto same = [](int, double v) { return v; };
  if (FWD) {
    coarse_pass<true>(S0, G0, 1, a, b, n, same);
    __syncthreads();
    coarse_pass<true>(S1, G1, G0, b, a, n, same);
  } else {
    coarse_pass<false>(S1, G1, G0, a, b, n, same);
    __syncthreads();
    coarse_pass<false>(S0, G0, 1, b, a, n, same);
  }
  __syncthreads();
  for (int q = tid; q < n; q += nth) {
    if (FWD) w[(int64_t)z * n + q] = a[q];
    else u[coarse_offset(C, q % G0, q / G0, z)] = (T)a[q];
  }
}
inline size_t coarse_planes_shmem(const CoarseDev& C) {
  const size_t G0 = coarse_nodes(C, 0), G1 = coarse_nodes(C, 1);
  return (2 * G0 * G1 + G0 * coarse_pitch((int)G0) + G1 * coarse_pitch((int)G1)) * sizeof(double);
}

// Columns of direction 2, COARSE_COLS per block: forward, scaled, back, in place in w.
constexpr int COARSE_COLS = 16;
__global__ void __launch_bounds__(256) coarse_columns_kernel(CoarseDev C, double* __restrict__ w, const int* active) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  if (inactive(active)) return;
  const int G0 = coarse_nodes(C, 0), G1 = coarse_nodes(C, 1), G = coarse_nodes(C, 2), np = G0 * G1;
  const int c0 = blockIdx.x * COARSE_COLS, nc = imin(COARSE_COLS, np - c0), n = G * COARSE_COLS;
  const int tid = threadIdx.x, nth = blockDim.x;
  double* a = reinterpret_cast<double*>(smem_raw);
  double* b = a + n;
  double* S = b + n;
  coarse_matrix(C.S[2], S, G);
  for (int q = tid; q < n; q += nth) {
    const int c = q % COARSE_COLS, z = q / COARSE_COLS;
    a[q] = c < nc ? w[(int64_t)z * np + c0 + c] : 0.0;
  }
  __syncthreads();
  coarse_pass<true>(S, G, COARSE_COLS, a, b, n, [&](int q, double v) {
    const int c = imin(c0 + q % COARSE_COLS, np - 1), z = q / COARSE_COLS;
    const double den = C.lam[0][c % G0] + C.lam[1][c / G0] + C.lam[2][z];
    return den != 0.0 ? v / den : 0.0;
  });
  __syncthreads();
  coarse_pass<false>(S, G, COARSE_COLS, b, a, n, [](int, double v) { return v; });
  __syncthreads();
  for (int q = tid; q < n; q += nth) {
    const int c = q % COARSE_COLS, z = q / COARSE_COLS;
    if (c < nc) w[(int64_t)z * np + c0 + c] = a[q];
  }
}
inline size_t coarse_columns_shmem(const CoarseDev& C) {
  const size_t G = coarse_nodes(C, 2);
  return (2 * G * COARSE_COLS + G * coarse_pitch((int)G)) * sizeof(double);
}

// out = f less its mean (out may be f), for grids that the one-block form could take but
// does not: the same order of the sum, so the same bits.
__global__ void __launch_bounds__(COARSE_THREADS) coarse_mean_kernel(CoarseDev C, const double* f, double* out,
                                                                     const int* active) {
  __shared__ double red[COARSE_THREADS / 64], mean;
  if (inactive(active)) return;
  const int G0 = coarse_nodes(C, 0), G1 = coarse_nodes(C, 1), n = G0 * G1 * coarse_nodes(C, 2);
  const auto at = [&](int q) {
    const int r = q / G0;
    return coarse_offset(C, q - r * G0, r % G1, r / G1);
  };
  double s = 0.0;
  for (int q = threadIdx.x; q < n; q += blockDim.x) s += f[at(q)];
  s = block_sum(s, red);
  if (threadIdx.x == 0) mean = s / (double)n;
  __syncthreads();
  for (int q = threadIdx.x; q < n; q += blockDim.x) out[at(q)] = f[at(q)] - mean;
}

// The form of a grid's coarse solve.  The one block has the rate of one compute unit, some
// 0.1 us per 1000 products of one way: it ends where the launches of the passes cost less
// (us, block / passes: 2D 22 x 22 elements, 170 k products, 21.0 / 21.4, 24 x 24, 221 k, 24.3 /
// 21.2; periodic, where the passes have two launches more for the means, 26 x 26, 281 k,
// 31.9 / 33.5, 28 x 28, 351 k, 38.8 / 34.5, 9^3, 315 k, 46.7 / 41).  Planes take 3D Dirichlet grids beyond 2048 unknowns
// (block / planes: 6^3 elements 14.7 / 13.0, 7^3 20 / 14) while a block's plane or columns
// are short beside the six launches (planes / passes: 16^3 25 / 28, 24 x 8 x 8 22 / 28, 4 x 4 x
// 35 26 / 27; beyond, 17^3 35 / 31, 20^3 44 / 32, 3 x 3 x 60 46 / 32), and the largest, whose
// passes stream the vector (30^3 92 / 96, 32 x 32 x 40 105 / 128).
enum CoarseForm { COARSE_BLOCK, COARSE_PLANES, COARSE_PASSES };
inline bool coarse_block_fits(const CoarseDev& C) { return coarse_block_shmem(C) <= COARSE_LDS; }
inline CoarseForm coarse_form(const CoarseDev& C, bool mean) {
  const int64_t G0 = coarse_nodes(C, 0), G1 = coarse_nodes(C, 1), G2 = coarse_nodes(C, 2), n = G0 * G1 * G2;
  const int64_t products = n * (G0 + G1 + (C.dim == 3 ? G2 : 0));
  const bool planes = C.dim == 3 && !mean && coarse_planes_shmem(C) <= COARSE_LDS &&
                      coarse_columns_shmem(C) <= COARSE_LDS &&
                      (n >= 200000 || (G0 * G1 * (G0 + G1) <= 70000 && 32 * G2 * G2 <= 130000));
  if (planes && n > 2048) return COARSE_PLANES;
  return coarse_block_fits(C) && products <= (mean ? 290000 : 200000) ? COARSE_BLOCK : (planes ? COARSE_PLANES : COARSE_PASSES);
}

}  // namespace dgmg
