// HIP kernels for gfx950 (MI355X): sum-factorised DG operator, Schwarz patch
// solves by fast diagonalisation, deterministic overlap summation, p-transfers.
//
// Vector layout (all kernels): element-major, element e = m1 + N1 (m2 + N2 m3),
// local node (k NP + j) NP + i, direction 1 fastest.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace dgmg {

constexpr int ipow(int b, int e) { return e == 0 ? 1 : b * ipow(b, e - 1); }
constexpr int imax(int a, int b) { return a > b ? a : b; }
constexpr int imin(int a, int b) { return a < b ? a : b; }
constexpr int round64(int a) { return (a + 63) / 64 * 64; }

constexpr int NUM_XCD = 8;  // MI355X: 8 accelerator complex dies, blocks dispatched round-robin

// Logical block index such that each XCD receives one contiguous range of
// logical blocks (neighbouring elements then share that XCD's L2).  The grid
// is launched with NUM_XCD * ceil(G / NUM_XCD) blocks; returns -1 for padding.
__device__ __forceinline__ int xcd_block(int G) {
  const int per = (G + NUM_XCD - 1) / NUM_XCD;
  const int b = blockIdx.x;
  const int lb = (b % NUM_XCD) * per + b / NUM_XCD;
  return lb < G ? lb : -1;
}
inline int xcd_grid(int G) { return NUM_XCD * ((G + NUM_XCD - 1) / NUM_XCD); }

enum { ECOEF_N = 8, E_TWO_DX = 0, E_HALF_DX, E_CL, E_CNL, E_BL, E_CR, E_CNR, E_BR };

template <class T>
struct DirDev {
  int N = 1, periodic = 0;
  int nl = 0;  // continuous levels: stored lattice nodes of the direction
  int n_ec = 0, n_fc = 0, nf = 0;
  const T* ecoef = nullptr;  // N * 8 (see ECOEF enum)
  const int* nbr = nullptr;  // N * 2
  const T* S_ec = nullptr;   // N * n_ec^2, row-major S[k][j]
  const T* ST_ec = nullptr;  // the transposes
  const T* lam_ec = nullptr;
  const T* w_ec = nullptr;
  const T* S_fc = nullptr;   // nf * n_fc^2
  const T* ST_fc = nullptr;
  const T* lam_fc = nullptr;
  const T* w_fc = nullptr;
  // offsets into the level vector of every patch position (-1 outside a
  // Dirichlet domain): N * n_ec and nf * n_fc
  const int* goff_ec = nullptr;
  const int* goff_fc = nullptr;
  // 3D tiles solved in LDS: the matrices S in the padded form of fdm3_image, and the
  // offsets of all positions of the direction in order (patch p's position o at
  // p step + o, step = the distance of consecutive patches)
  const T* img_ec = nullptr;
  const T* img_fc = nullptr;
  const int* gp_ec = nullptr;
  const int* gp_fc = nullptr;
};

template <class T>
struct LevelDev {
  int dim = 3, P = 1, NP = 2, NO = 0, NPc = 0;
  int se = 0;  // 1: continuous spectral-element level (lattice vectors)
  int n_elem = 0;
  int64_t n_dof = 0;
  const T* Ls = nullptr;   // NP*NP
  const T* D = nullptr;    // NP*NP, D[i*NP+k] = phi_k'(eta_i)
  const T* rho = nullptr;  // NP
  const T* J = nullptr;    // NP x NPc interpolation from the coarser level
  const int* active = nullptr;  // batched solves: the kernels return at once when *active == 0
  DirDev<T> dir[3];
};

__device__ __forceinline__ bool inactive(const int* flag) { return flag != nullptr && *flag == 0; }

// Patches of one launch: per direction the patch indices start + stride * k,
// k = 0 .. count - 1 (the additive sweeps take all of them: start 0, stride 1;
// a colour class of the multiplicative smoothers takes every k-th).
struct PatchLat {
  int start[3] = {0, 0, 0};
  int stride[3] = {1, 1, 1};
};

// Layout of the patch buffer.  K > 1: strips of K patches along direction 1 whose
// tiles, `step` planes apart, are summed where they overlap (one tile of
// (K - 1) step + len planes per strip); K is a power of two.  swp: tiles are stored plane by plane of
// direction 1, [o1][o2][o0] (fdm3_kernel), instead of [o2][o1][o0].
struct PatchBuf {
  int K = 1, step = 0, swp = 0;
};

constexpr size_t LDS_BYTES = 160 * 1024;  // gfx950 LDS per workgroup

// A len x len matrix in LDS: rows padded with zeros to the operands' blocks, and a
// pitch of 2 (mod 16) so that the four rows and four columns of an operand block lie
// on distinct banks, read as M or as its transpose.  The patch matrices are kept in
// device memory in this form (fdm3_image values each): a block copies them in 16-byte
// pieces without index arithmetic.  FP32 rows beyond 32 are not padded (33 would become
// 48, and three such matrices do not fit the LDS beside a 33^3 tile): their readers
// mask what lies outside the matrix.
template <class T>
constexpr bool fdm3_padded(int len) {
  return sizeof(T) == 8 || len <= 32;
}
template <class T>
constexpr int fdm3_rows(int len) {
  return sizeof(T) == 8 ? (len + 3) / 4 * 4 : (fdm3_padded<T>(len) ? (len + 15) / 16 * 16 : len);
}
template <class T>
constexpr int fdm3_pitch(int len) {
  return fdm3_rows<T>(len) + 2;
}
template <class T>
constexpr int fdm3_image(int len) {
  constexpr int piece = 16 / (int)sizeof(T);
  return (fdm3_rows<T>(len) * fdm3_pitch<T>(len) + piece - 1) / piece * piece;
}

// Work list of a batched launch: one kernel over the work of many grids.  The
// launch's logical blocks are split into consecutive ranges, range g
// (starts[g] <= b < starts[g + 1], g < ng) doing grid g's blocks with the
// arguments descs[g] (device arrays; the grid index is uniform per block, so
// these reads are scalar loads).
template <class A>
struct BatchList {
  const A* descs = nullptr;
  const int* starts = nullptr;
  int ng = 0;
};

// Arguments of logical block b of a batched launch, copied into the block's
// LDS slot `args` (the kernels index their argument structs with run-time
// direction indices: from LDS that stays a plain LDS read, from a local copy it
// would go through scratch memory); returns the block's index within its grid.
// Called by every thread of the block.
template <class A>
__device__ __forceinline__ int batch_pick(const BatchList<A>& bl, int b, A* args) {
  static_assert(sizeof(A) % sizeof(int) == 0, "argument struct of whole words");
  const int* __restrict__ st = bl.starts;
  int lo = 0, hi = bl.ng - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (st[mid] <= b) lo = mid;
    else hi = mid - 1;
  }
  lo = __builtin_amdgcn_readfirstlane(lo);
  const int* __restrict__ src = reinterpret_cast<const int*>(bl.descs + lo);
  int* dst = reinterpret_cast<int*>(args);
  for (int i = threadIdx.x; i < (int)(sizeof(A) / sizeof(int)); i += blockDim.x) dst[i] = src[i];
  __syncthreads();
  return b - st[lo];
}

// ---------------------------------------------------------------- block reduction
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Deterministic block sum (fixed shuffle tree then fixed order over waves).
__device__ __forceinline__ double block_sum(double v, double* red) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) red[w] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0) {
    const int nw = (blockDim.x + 63) >> 6;
    for (int i = 0; i < nw; ++i) s += red[i];
  }
  return s;  // valid in thread 0
}

// Quotient by a divisor known to the host: m = ceil(2^32 / d) where the product
// fits (every n up to n_max is then exact), 0 otherwise.
inline uint32_t div_magic(int64_t n_max, int d) {
  return n_max * d < (int64_t(1) << 32) && d > 1 ? (uint32_t)(((uint64_t(1) << 32) + d - 1) / d) : 0;
}
__device__ __forceinline__ int div_by(int n, int d, uint32_t m) {
  return m ? (int)__umulhi((uint32_t)n, m) : (d == 1 ? n : n / d);
}

// A kernel-argument pointer pinned in scalar registers: selecting between such
// values per lane stays a register select instead of becoming a per-lane load
// from the argument segment (which would make the loads behind it dependent).
template <class P>
__device__ __forceinline__ P* sgpr_ptr(P* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<P*>(((uint64_t)hi << 32) | lo);
}

// Move n <= N values with every load of a thread issued before any of its
// stores (a plain strided loop waits for each load before the next one
// starts).  NT is the block size; ld(e) reads element e (called with e < n
// only), st(e, v) writes it.
template <class T, int NT, int N, class Ld, class St>
__device__ __forceinline__ void staged_copy(Ld ld, St st, int n = N) {
  constexpr int C = (N + NT - 1) / NT;
  const int tid = threadIdx.x;
  T v[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int e = tid + c * NT;
    v[c] = ld(e < n ? e : n - 1);
  }
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int e = tid + c * NT;
    if (e < n) st(e, v[c]);
  }
}

// ================================================================ FDM patch solve
// v / d for d > 0 of moderate magnitude (sums of patch eigenvalues): hardware
// reciprocal estimate (FP64: to about 2^-26, refined by one Newton-Raphson step), then
// one residual correction of the quotient, which squares the estimate's error again
// (within an ulp of the rounded quotient).
__device__ __forceinline__ double div_nr(double v, double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = fma(fma(-d, r, 1.0), r, r);
  const double q = v * r;
  return fma(fma(-d, q, v), r, q);
}
__device__ __forceinline__ float div_nr(float v, float d) {
  float r = __builtin_amdgcn_rcpf(d);
  r = fmaf(fmaf(-d, r, 1.0f), r, r);
  const float q = v * r;
  return fmaf(fmaf(-d, q, v), r, q);
}
// 2D tiles and short 3D tiles (fdm_short; the others: kernels_fdm3.hpp), one patch per
// block.  The LDS tile keeps the normal direction fastest: tile[(l2 * NL + l1) * NAP + a],
// NAP = NA rounded up to an odd pitch so that the lines of the fastest pass spread over the
// LDS banks.  NA = 2P for a face-centred patch (the element-centred size otherwise),
// NL = NP + 2 N_O.  Passes over longer lines run on the matrix cores: the lines of the
// tile are the M dimension (blocks of 16), the 1D eigenbasis is the B operand held in
// registers, and each wave overwrites its line blocks in place; short lines go to the VALU,
// a line per thread.
template <int NA, int NL, int DIM>
constexpr int fdm_tile() {
  return NA * ipow(NL, DIM - 1);
}
template <int NA>
constexpr int fdm_pitch() {
  return NA % 2 == 0 ? NA + 1 : NA;
}
template <int NA, int NL, int DIM>
constexpr int fdm_tile_padded() {
  return fdm_pitch<NA>() * ipow(NL, DIM - 1);
}
// Lines up to this length are contracted on the VALU, longer ones on the
// matrix cores (fdm_pass_any).
constexpr int FDM_VALU_MAXLEN = 9;
// Default block size of a patch solve (the autotuner may choose another): a
// thread per line of the longest pass, at most 256.
template <int NA, int NL, int DIM>
constexpr int fdm_threads() {
  return imin(256, round64(imax(ipow(NL, DIM - 1), NA * ipow(NL, DIM - 2))));
}
template <class T, int NA, int NL, int DIM>
constexpr size_t fdm_shmem() {
  return (size_t)fdm_tile_padded<NA, NL, DIM>() * sizeof(T);
}

// 16x16x4 matrix-core contraction (v_mfma_{f64,f32}_16x16x4): A[i][k] comes from lane
// i + 16k and B[k][j] from lane j + 16k.  Result register r of lane l holds
// D[row(l / 16, r)][l % 16] with row = l/16 + 4r for f64 and 4 (l/16) + r for f32
// (layouts checked on gfx950 with one-hot operands).
template <class T>
struct Mfma;
template <>
struct Mfma<double> {
  typedef double acc_t __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc_t op(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lk, int r) { return lk + 4 * r; }
};
template <>
struct Mfma<float> {
  typedef float acc_t __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc_t op(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lk, int r) { return 4 * lk + r; }
};

// Line start inside the padded tile for contraction dimension TD.
template <int NA, int NL, int TD>
__device__ __forceinline__ int fdm_line_base(int line) {
  constexpr int NAP = fdm_pitch<NA>();
  if (TD == 0) return line * NAP;
  const int a = line % NA, q = line / NA;
  return TD == 1 ? q * NAP * NL + a : q * NAP + a;
}

// The 1D matrix of a contraction (row-major LEN x LEN) in registers: lane
// (li, lk) = (lane % 16, lane / 16) holds B[4 ks + lk][16 nb + li], i.e. the
// A operand (B^T)[16 nb + li][4 ks + lk] of the transposed product.
template <class T, int LEN>
struct BOp {
  static constexpr int KS = (LEN + 3) / 4, NB = (LEN + 15) / 16;
  T b[NB][KS];
  __device__ __forceinline__ void load(const T* __restrict__ Bm) {
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int k = 4 * ks + lk, j = nb * 16 + li;
        // unconditional load at a valid index, zero outside the matrix (no branch)
        const T v = Bm[imin(k, LEN - 1) * LEN + imin(j, LEN - 1)];
        b[nb][ks] = (k < LEN && j < LEN) ? v : T(0);
      }
  }
};

// One contraction pass over tile dimension TD: every line v (length LEN) is
// replaced by B^T v, i.e. out_j = sum_k B[k][j] v_k.  The lines form the M
// dimension in blocks of 16; each wave owns whole blocks, reading a block
// (A operand) completely before writing it back in place.
struct NoPost {
  template <class T>
  __device__ __forceinline__ T operator()(int, int, T v) const { return v; }
};

// post(line, j, value) maps each result before it is stored (e.g. the
// eigenvalue scaling fused into the last forward pass).
// No lane-dependent branches: loads past the end of a line or of the line set
// read a valid element instead (the matrix operand is zero for k >= LEN, and
// results of lines past the set are discarded), and stores of rows j >= LEN or
// of lines past the set go to the lane's slot of `trash` (64 values, dead
// storage) instead of being masked.
template <class T, int NA, int NL, int DIM, int TD, class Post>
__device__ __forceinline__ void fdm_pass(T* __restrict__ tile, T* __restrict__ trash,
                                         const BOp<T, TD == 0 ? NA : NL>& B, Post post) {
  // Product D = B^T V^T: the A operand is B^T (held as B.b), the B operand the
  // lines; lane (li, lk) then owns output column li = its own line, rows
  // j = 16 nb + row(lk, r), so results go back along the line it loaded.
  constexpr int NAP = fdm_pitch<NA>();
  constexpr int LEN = TD == 0 ? NA : NL;
  constexpr int LINES = TD == 0 ? ipow(NL, DIM - 1) : NA * ipow(NL, DIM - 2);
  constexpr int STRIDE = TD == 0 ? 1 : (TD == 1 ? NAP : NAP * NL);
  constexpr int KS = BOp<T, LEN>::KS, NB = BOp<T, LEN>::NB, MB = (LINES + 15) / 16;
  using M = Mfma<T>;
  // the wave index is uniform over the wave: keeping it scalar makes the block
  // loop a scalar loop
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = blockDim.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
  for (int mb = wave; mb < MB; mb += nw) {
    const int line = mb * 16 + li;
    const bool lv = line < LINES;
    const int lc = imin(line, LINES - 1);
    const int base = fdm_line_base<NA, NL, TD>(lc);
    typename M::acc_t acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = typename M::acc_t{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int k = imin(4 * ks + lk, LEN - 1);
      const T a = tile[base + k * STRIDE];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[nb] = M::op(B.b[nb][ks], a, acc[nb]);
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int j = nb * 16 + M::row(lk, r);
        const bool ok = lv && j < LEN;
        const int jc = imin(j, LEN - 1);
        T* dst = ok ? tile + base + jc * STRIDE : trash + lane;
        *dst = post(lc, jc, acc[nb][r]);
      }
  }
}

template <class T, int NA, int NL, int DIM, int TD, class Post = NoPost>
__device__ __forceinline__ void fdm_pass(T* __restrict__ tile, T* __restrict__ trash, const T* __restrict__ Bm,
                                         Post post = Post()) {
  BOp<T, TD == 0 ? NA : NL> B;
  B.load(Bm);
  fdm_pass<T, NA, NL, DIM, TD, Post>(tile, trash, B, post);
}

// VALU form of a contraction pass: one line per thread, out_j = sum_k B[k][j] v_k,
// reading BT = B^T (row-major, so the coefficients of one output are one
// contiguous row) through scalar loads: the matrix is uniform over the block.
// Exact line lengths: FP64 vector FMA and FP64 MFMA have the same peak rate on
// gfx950, and the matrix-core form pads lengths like 13 to 16 in both the K
// and N dimensions (66 % useful work), so short lateral lines are cheaper here.
// Same post(line, j, value) contract as fdm_pass.
// Rows of the matrix per step of the VALU pass: the largest divisor R of LEN
// with R LEN values within 32 FP64 (64 FP32) SGPR pairs / SGPRs.
template <class T, int LEN>
constexpr int fdm_valu_rows() {
  constexpr int cap = sizeof(T) == 8 ? 32 : 64;
  int best = 1;
  for (int r = 1; r <= LEN; ++r)
    if (LEN % r == 0 && r * LEN <= cap) best = r;
  return best;
}

template <class T, int NA, int NL, int DIM, int TD, class Post = NoPost>
__device__ __forceinline__ void fdm_pass_valu(T* __restrict__ tile, const T* __restrict__ BTm,
                                              Post post = Post()) {
  constexpr int NAP = fdm_pitch<NA>();
  constexpr int LEN = TD == 0 ? NA : NL;
  constexpr int LINES = TD == 0 ? ipow(NL, DIM - 1) : NA * ipow(NL, DIM - 2);
  constexpr int STRIDE = TD == 0 ? 1 : (TD == 1 ? NAP : NAP * NL);
  using CT = const __attribute__((address_space(4))) T;
  CT* __restrict__ BT = (CT*)BTm;
  constexpr int R = fdm_valu_rows<T, LEN>();
  for (int line = threadIdx.x; line < LINES; line += blockDim.x) {
    const int base = fdm_line_base<NA, NL, TD>(line);
    T v[LEN];
#pragma unroll
    for (int k = 0; k < LEN; ++k) v[k] = tile[base + k * STRIDE];
    // R rows of BT per step: R independent accumulation chains, one scalar
    // load group per step, at most 32 FP64 (64 FP32) matrix values in SGPRs
#pragma unroll 1
    for (int j0 = 0; j0 < LEN; j0 += R) {
      const int ju = __builtin_amdgcn_readfirstlane(j0);
      T acc[R];
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r] = 0;
#pragma unroll
      for (int k = 0; k < LEN; ++k)
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] += BT[(ju + r) * LEN + k] * v[k];
#pragma unroll
      for (int r = 0; r < R; ++r) tile[base + (j0 + r) * STRIDE] = post(line, j0 + r, acc[r]);
    }
  }
}

// Contraction pass of tile dimension TD on the unit that suits its length:
// lines up to FDM_VALU_MAXLEN long go to the VALU (the matrix-core form
// would pad a length-9 line to 12 x 16, 42 % useful work), longer ones to the
// matrix cores (measured on an MI355X: length 13 lateral passes on the VALU made
// the 16 x 13 x 13 patch solve 9 % slower, every pass on the VALU 35 %).
template <class T, int NA, int NL, int DIM, int TD, class Post = NoPost>
__device__ __forceinline__ void fdm_pass_any(T* __restrict__ tile, T* __restrict__ trash, const T* __restrict__ Bm,
                                             const T* __restrict__ BTm, Post post = Post()) {
  constexpr int LEN = TD == 0 ? NA : NL;
  constexpr bool VALU = LEN <= FDM_VALU_MAXLEN;
  if constexpr (VALU) fdm_pass_valu<T, NA, NL, DIM, TD, Post>(tile, BTm, post);
  else fdm_pass<T, NA, NL, DIM, TD, Post>(tile, trash, Bm, post);
}

// Tile geometry of one sweep kind, all compile-time: ND = normal direction of a
// face-centred patch (-1: element-centred).  Grid-natural order has direction 0
// fastest with lengths L0, L1, L2; the LDS tile keeps the normal direction
// fastest: tile[(l2 NL + l1) NAP + a].
template <int DIM, int ND, int NA, int NL>
struct FdmShape {
  static constexpr int L0 = ND == 0 ? NA : NL;
  static constexpr int L1 = ND == 1 ? NA : NL;
  static constexpr int L2 = DIM == 3 ? (ND == 2 ? NA : NL) : 1;
  static constexpr int TS = L0 * L1 * L2;
  static constexpr int NROW = L1 * L2;  // rows of the grid-natural order (fixed o1, o2)
  static constexpr int NAP = fdm_pitch<NA>();
  // tile stride of direction 0 (the normal / fastest tile dimension unless ND > 0)
  static constexpr int C0 = ND <= 0 ? 1 : NAP;
  // grid direction of tile dimension t (t = 0: the normal / fastest one)
  static constexpr int gd(int t) { return ND <= 0 ? t : (t == 0 ? ND : (t <= ND ? t - 1 : t)); }
  static __device__ __forceinline__ int tpos(int o0, int o1, int o2) {
    const int o[3] = {o0, o1, o2};
    return ((DIM == 3 ? o[gd(2)] * NL : 0) + o[gd(1)]) * NAP + o[gd(0)];
  }
};

// 3D tiles that fdm_kernel solves in sweeps of many patches: lines of up to 7 values (in FP64
// not the shortest, 3 x 3 to 4 x 4), where the matrix cores' operands (blocks of 4 lines and 4 values in FP64,
// 16 lines and 16 values in FP32) are mostly padding.  Whole sweeps, kernels_fdm3.hpp / here,
// us: 5 x 5 x 5 on 6156 patches FP64 16.6 / 12.4, FP32 15.1 / 9.8, on 44100 56 / 49 and 52 / 38;
// 6 x 6 x 6 on 20412 41 / 34 and 37 / 26; 8 x 5 x 5 on 9702 23 / 21 and 22 / 15; 7 x 7 x 7 on
// 16250 without strips FP64 58 / 40, FP32 47 / 28, on 9702 with strips FP64 27 / 31, FP32 25 /
// 21; 4 x 4 x 4 on 20412 FP64 17 / 21, FP32 19 / 15; 6 x 4 x 4 on 6156 FP64 14.1 / 11.7.  With
// fewer patches the chain of passes is the time: 810 patches of 5 x 5 x 5 6.1 / 6.3, 1452 of
// 6 x 6 x 6 FP64 8.6 / 8.6, of 7 x 7 x 7 FP64 10.0 / 13.8 (2940: 15.4 / 14.4).  strips: patches can share planes along direction 1.
template <class T>
constexpr bool fdm_short(int NA, int NL) {
  return NA <= 8 && NL <= 7 && (sizeof(T) == 4 || NL >= 5 || NA >= 6);
}
template <class T>
bool fdm_short_fits(int NA, int NL, int64_t patches, bool strips) {
  if (sizeof(T) == 8 && NL == 7) return fdm_short<T>(NA, NL) && !strips && patches >= 2400;
  return fdm_short<T>(NA, NL) && patches >= 1200;
}

template <class T>
struct FdmArgs {
  LevelDev<T> L;
  const T* r = nullptr;  // residual (level vector)
  T* out = nullptr;      // weighted corrections, one tile per patch of the launch
  int npx = 1, npy = 1, npz = 1;
  PatchLat lat;
};

// BATCH: the arguments come from the work list bl (ntot logical blocks in all)
template <class T, int DIM, int NA, int NL, int ND, bool BATCH = false>
__global__ void __launch_bounds__(512) fdm_kernel(FdmArgs<T> a0, BatchList<FdmArgs<T>> bl, int ntot) {
  static_assert(DIM == 2 || fdm_short<T>(NA, NL), "other 3D tiles: fdm3_kernel");
  using S = FdmShape<DIM, ND, NA, NL>;
  constexpr int TS = S::TS;
  constexpr int NMAX = imax(NA, NL);
  constexpr int GU = 4;  // elements gathered per thread before their LDS stores (loads in flight)
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* tile = reinterpret_cast<T*>(smem_raw);
  __shared__ int goff[3][NMAX];  // offsets into the level vector (< 2^31 unknowns), -1 outside
  __shared__ T wv[3][NMAX];
  __shared__ T lv[3][NMAX];
  // rowoff is dead once the gather is done: the contraction passes use it as
  // their store trash (64 values)
  __shared__ __align__(8) int rowoff[imax(S::NROW, 64 * (int)sizeof(T) / (int)sizeof(int))];
  __shared__ int rowpos[S::NROW];
  __shared__ __align__(16) int sargs_raw[BATCH ? sizeof(FdmArgs<T>) / sizeof(int) : 1];
  FdmArgs<T>* sargs = reinterpret_cast<FdmArgs<T>*>(sargs_raw);
  const FdmArgs<T>* ap;
  int pid;
  if constexpr (BATCH) {
    const int b = xcd_block(ntot);
    if (b < 0) return;
    pid = batch_pick(bl, b, sargs);
    ap = sargs;
  } else {
    pid = xcd_block(a0.npx * a0.npy * a0.npz);
    if (pid < 0) return;
    ap = &a0;
  }
  const LevelDev<T>& L = ap->L;
  const T* __restrict__ r = ap->r;
  T* __restrict__ out = ap->out;
  const int npx = ap->npx, npy = ap->npy;
  const PatchLat& lat = ap->lat;
  if (inactive(L.active)) return;
  const int tid = threadIdx.x, nth = blockDim.x;
  int p[3];
  p[0] = lat.start[0] + lat.stride[0] * (pid % npx);
  p[1] = lat.start[1] + lat.stride[1] * (DIM == 3 ? (pid / npx) % npy : pid / npx);
  p[2] = DIM == 3 ? lat.start[2] + lat.stride[2] * (pid / (npx * npy)) : 0;
  const int* go[3] = {nullptr, nullptr, nullptr};
  const T* wg[3] = {nullptr, nullptr, nullptr};
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    const DirDev<T>& dd = L.dir[d];
    const bool fc = d == ND;
    const int len = fc ? NA : NL;
    go[d] = fc ? dd.goff_fc + p[d] * NA : dd.goff_ec + p[d] * NL;
    wg[d] = fc ? dd.w_fc + p[d] * NA : dd.w_ec + p[d] * NL;
    const T* lam = fc ? dd.lam_fc + p[d] * NA : dd.lam_ec + p[d] * NL;
    for (int o = tid; o < len; o += nth) {
      goff[d][o] = go[d][o];
      wv[d][o] = wg[d][o];
      lv[d][o] = lam[o];
    }
  }
  // per row (o1, o2) of the grid-natural order: its offset in the level vector (-1 outside a
  // Dirichlet domain) and its tile position
  for (int rw = tid; rw < S::NROW; rw += nth) {
    const int o1 = rw % S::L1, o2 = rw / S::L1;
    const int g1 = go[1][o1], g2 = DIM == 3 ? go[2][o2] : 0;
    rowoff[rw] = (g1 | g2) < 0 ? -1 : g1 + g2;
    rowpos[rw] = S::tpos(0, o1, o2);
  }
  // 1D matrices of each tile dimension: forward t_j = sum_k S_kj r_k uses S,
  // backward u_k = sum_j S_kj t_j uses S^T (both row-major)
  const T* fwd[3] = {nullptr, nullptr, nullptr};
  const T* bwd[3] = {nullptr, nullptr, nullptr};
#pragma unroll
  for (int t = 0; t < DIM; ++t) {
    const int d = S::gd(t);
    const DirDev<T>& dd = L.dir[d];
    if (d == ND) {
      fwd[t] = dd.S_fc + (int64_t)p[d] * NA * NA;
      bwd[t] = dd.ST_fc + (int64_t)p[d] * NA * NA;
    } else {
      fwd[t] = dd.S_ec + (int64_t)p[d] * NL * NL;
      bwd[t] = dd.ST_ec + (int64_t)p[d] * NL * NL;
    }
  }
  __syncthreads();
  // gather R_s r in grid-natural order (coalesced global reads); GU loads are
  // issued before their LDS stores; positions outside a Dirichlet domain read
  // r[0] and store 0
  constexpr bool G2D = S::L0 == 16;  // shorter rows would idle lanes (measured slower)
  if constexpr (G2D) {
    // lanes in groups of 16 along direction 0 (o0 = tid % 16), rows in steps of nth / 16
    const int o0 = tid & 15, rstep = nth >> 4;
    const bool colok = o0 < S::L0;
    const int oc = colok ? o0 : 0;
    const int g0 = goff[0][oc], pc = oc * S::C0;
    for (int rw0 = tid >> 4; rw0 < S::NROW; rw0 += GU * rstep) {
      T v[GU];
      int pos[GU];
#pragma unroll
      for (int u = 0; u < GU; ++u) {
        const int rw = rw0 + u * rstep;
        const bool in = colok && rw < S::NROW;
        const int rwc = rw < S::NROW ? rw : 0;
        const int ro = rowoff[rwc];
        const bool ok = in && (g0 | ro) >= 0;
        v[u] = r[ok ? g0 + ro : 0];
        v[u] = ok ? v[u] : T(0);
        pos[u] = in ? rowpos[rwc] + pc : -1;
      }
#pragma unroll
      for (int u = 0; u < GU; ++u)
        if (pos[u] >= 0) tile[pos[u]] = v[u];
    }
  } else {
    for (int q0 = tid; q0 < TS; q0 += GU * nth) {
      T v[GU];
      int pos[GU];
#pragma unroll
      for (int u = 0; u < GU; ++u) {
        const int q = q0 + u * nth;
        const int qq = q < TS ? q : 0;
        const int o0 = qq % S::L0, rw = qq / S::L0;
        const int g0 = goff[0][o0], ro = rowoff[rw];
        const bool ok = q < TS && (g0 | ro) >= 0;
        v[u] = r[ok ? g0 + ro : 0];
        v[u] = ok ? v[u] : T(0);
        pos[u] = q < TS ? rowpos[rw] + o0 * S::C0 : -1;
      }
#pragma unroll
      for (int u = 0; u < GU; ++u)
        if (pos[u] >= 0) tile[pos[u]] = v[u];
    }
  }
  __syncthreads();
  T* trash = reinterpret_cast<T*>(rowoff);
  // the last forward pass divides each result by the sum of the 1D eigenvalues of its tile
  // position: line = a + NA l1 and j = l2 (2D: line = a, j = l1)
  const auto scale = [&](int line, int j, T v) -> T {
    T den = lv[S::gd(0)][line % NA] + lv[S::gd(1)][DIM == 3 ? line / NA : j];
    if constexpr (DIM == 3) den += lv[S::gd(2)][j];
    return div_nr(v, den);
  };
  fdm_pass_any<T, NA, NL, DIM, 0>(tile, trash, fwd[0], bwd[0]);
  __syncthreads();
  if constexpr (DIM == 3) {
    fdm_pass_any<T, NA, NL, DIM, 1>(tile, trash, fwd[1], bwd[1]);
    __syncthreads();
  }
  fdm_pass_any<T, NA, NL, DIM, DIM - 1>(tile, trash, fwd[DIM - 1], bwd[DIM - 1], scale);
  __syncthreads();
  fdm_pass_any<T, NA, NL, DIM, DIM - 1>(tile, trash, bwd[DIM - 1], fwd[DIM - 1]);
  __syncthreads();
  if constexpr (DIM == 3) {
    fdm_pass_any<T, NA, NL, DIM, 1>(tile, trash, bwd[1], fwd[1]);
    __syncthreads();
  }
  fdm_pass_any<T, NA, NL, DIM, 0>(tile, trash, bwd[0], fwd[0]);
  __syncthreads();
  // weighted result w_s (.) Delta u_s in grid-natural order
  const auto row_w = [&](int rw) -> T {
    if constexpr (DIM == 3) return wv[1][rw % S::L1] * wv[2][rw / S::L1];
    else return wv[1][rw];
  };
  T* dst = out + (int64_t)pid * TS;
  if constexpr (G2D) {
    const int o0 = tid & 15, rstep = nth >> 4;
    if (o0 < S::L0) {
      const T w0 = wv[0][o0];
      const int pc = o0 * S::C0;
      for (int rw = tid >> 4; rw < S::NROW; rw += rstep) dst[rw * S::L0 + o0] = (w0 * row_w(rw)) * tile[rowpos[rw] + pc];
    }
  } else {
    for (int q = tid; q < TS; q += nth) {
      const int o0 = q % S::L0, rw = q / S::L0;
      dst[q] = (wv[0][o0] * row_w(rw)) * tile[rowpos[rw] + o0 * S::C0];
    }
  }
}

template <class T, int DIM, int NA, int NL, int ND, bool BATCH>
void fdm_launch_nd(const FdmArgs<T>& a, const BatchList<FdmArgs<T>>& bl, int nlog, int th, size_t shm,
                   hipStream_t s) {
  if (shm > 65536)
    (void)hipFuncSetAttribute((const void*)fdm_kernel<T, DIM, NA, NL, ND, BATCH>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
  hipLaunchKernelGGL((fdm_kernel<T, DIM, NA, NL, ND, BATCH>), dim3(xcd_grid(nlog)), dim3(th), shm, s, a, bl, nlog);
}

// The same solve for sweeps of few patches, where one patch's chain of operations is the
// time: a thread per node of the tile (or a few), matrices and tile in LDS, four passes of
// one product row each.  256 patches, FP64: 23 x 23 10.4 -> 7.0 us, 9 x 9 6.3 -> 2.9 us
// (a launch alone: 2 us).  Its LDS reads (two per product) bound it when the GPU is full,
// where the matrix cores of fdm_kernel win: 1024 patches of 23 x 23 11.7 against 19.2 us.
// The two meet at 484 (FP64) and 961 (FP32) patches of 23 x 23, 480 of 24 x 19, 1100 and
// 2300 of 13 x 13, beyond 4096 of 9 x 9: at FDM2_BYTES of tiles or above.
constexpr int64_t FDM2_BYTES = 3 << 19;
constexpr int FDM2_NODES = 800;  // largest tile (a thread takes at most two nodes)
template <int NA, int NL, int ND>
constexpr int fdm2_threads() {
  return imin(512, round64((ND == 0 ? NA : NL) * (ND == 1 ? NA : NL)));
}
template <class T, int NA, int NL, int ND, bool BATCH = false>
__global__ void __launch_bounds__((fdm2_threads<NA, NL, ND>()))
    fdm2_kernel(FdmArgs<T> a0, BatchList<FdmArgs<T>> bl, int ntot) {
  constexpr int L0 = ND == 0 ? NA : NL, L1 = ND == 1 ? NA : NL, N = L0 * L1, TH = fdm2_threads<NA, NL, ND>();
  constexpr int P0 = L0 | 1, P1 = L1 | 1, C = (N + TH - 1) / TH;  // odd pitches: rows and columns on distinct banks
  __shared__ T S0[L0 * P0], S1[L1 * P1], A[L1 * P0], B[L1 * P0], sl[L0 + L1], sw[L0 + L1];
  __shared__ __align__(16) int sargs_raw[BATCH ? sizeof(FdmArgs<T>) / sizeof(int) : 1];
  const FdmArgs<T>* ap;
  int pid = 0;
  if constexpr (BATCH) {
    const int b = xcd_block(ntot);
    if (b < 0) return;
    FdmArgs<T>* sargs = reinterpret_cast<FdmArgs<T>*>(sargs_raw);
    pid = batch_pick(bl, b, sargs);
    ap = sargs;
  } else {
    ap = &a0;
  }
  // every argument into scalar registers by one group of loads
  const auto uni = [](int v) { return BATCH ? __builtin_amdgcn_readfirstlane(v) : v; };
  const auto ptr = [](auto* q) { return BATCH ? sgpr_ptr(q) : q; };
  const DirDev<T>&d0 = ap->L.dir[0], &d1 = ap->L.dir[1];
  const T *pS0 = ptr(ND == 0 ? d0.S_fc : d0.S_ec), *pS1 = ptr(ND == 1 ? d1.S_fc : d1.S_ec);
  const T *pl0 = ptr(ND == 0 ? d0.lam_fc : d0.lam_ec), *pl1 = ptr(ND == 1 ? d1.lam_fc : d1.lam_ec);
  const T *pw0 = ptr(ND == 0 ? d0.w_fc : d0.w_ec), *pw1 = ptr(ND == 1 ? d1.w_fc : d1.w_ec);
  const int *pg0 = ptr(ND == 0 ? d0.goff_fc : d0.goff_ec), *pg1 = ptr(ND == 1 ? d1.goff_fc : d1.goff_ec);
  const T* pr = ptr(ap->r);
  T* po = ptr(ap->out);
  const int* act = ptr(ap->L.active);
  int npx = uni(ap->npx), npy = uni(ap->npy), st0 = uni(ap->lat.start[0]), st1 = uni(ap->lat.start[1]);
  int sr0 = uni(ap->lat.stride[0]), sr1 = uni(ap->lat.stride[1]);
  if constexpr (!BATCH) {
    asm volatile("" : "+s"(pS0), "+s"(pS1), "+s"(pl0), "+s"(pl1), "+s"(pw0), "+s"(pw1), "+s"(pg0), "+s"(pg1), "+s"(pr),
                 "+s"(po), "+s"(act), "+s"(npx), "+s"(npy), "+s"(st0));
    asm volatile("" : "+s"(st1), "+s"(sr0), "+s"(sr1));
    pid = xcd_block(npx * npy);
    if (pid < 0) return;
  }
  using G = const __attribute__((address_space(1))) T;  // global memory
  using GI = const __attribute__((address_space(1))) int;
  if (act != nullptr && *(GI*)act == 0) return;
  pid = uni(pid);
  const int tid = threadIdx.x, p0 = st0 + sr0 * (pid % npx), p1 = st1 + sr1 * (pid / npx);
  G *gS0 = (G*)pS0 + (int64_t)p0 * L0 * L0, *gS1 = (G*)pS1 + (int64_t)p1 * L1 * L1, *r = (G*)pr;
  GI *g0 = (GI*)pg0 + p0 * L0, *g1 = (GI*)pg1 + p1 * L1;
  // nodes q = tid + c TH: position (x, y); positions outside a Dirichlet domain read r[0] and take 0
  int x[C], y[C], off[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int q = imin(tid + c * TH, N - 1);
    y[c] = q / L0;
    x[c] = q - y[c] * L0;
    const int a = g0[x[c]], b = g1[y[c]];
    off[c] = (a | b) < 0 ? -1 : a + b;
  }
  constexpr int M0 = (L0 * L0 + TH - 1) / TH, M1 = (L1 * L1 + TH - 1) / TH;
  T m0[M0], m1[M1];
#pragma unroll
  for (int c = 0; c < M0; ++c) m0[c] = gS0[imin(tid + c * TH, L0 * L0 - 1)];
#pragma unroll
  for (int c = 0; c < M1; ++c) m1[c] = gS1[imin(tid + c * TH, L1 * L1 - 1)];
  for (int q = tid; q < L0 + L1; q += TH) {
    const bool f = q < L0;
    const int64_t at = f ? (int64_t)p0 * L0 + q : (int64_t)p1 * L1 + (q - L0);
    sl[q] = f ? ((G*)pl0)[at] : ((G*)pl1)[at];
    sw[q] = f ? ((G*)pw0)[at] : ((G*)pw1)[at];
  }
  T v[C];
#pragma unroll
  for (int c = 0; c < C; ++c) v[c] = r[off[c] < 0 ? 0 : off[c]];
#pragma unroll
  for (int c = 0; c < M0; ++c) {
    const int q = tid + c * TH;
    if (q < L0 * L0) S0[q / L0 * P0 + q % L0] = m0[c];
  }
#pragma unroll
  for (int c = 0; c < M1; ++c) {
    const int q = tid + c * TH;
    if (q < L1 * L1) S1[q / L1 * P1 + q % L1] = m1[c];
  }
  const auto each = [&](auto f) {
#pragma unroll
    for (int c = 0; c < C; ++c)
      if (c + 1 < C || N % TH == 0 || tid + c * TH < N) f(c, x[c], y[c]);
  };
  each([&](int c, int i, int j) { A[j * P0 + i] = off[c] < 0 ? T(0) : v[c]; });
  __syncthreads();
  each([&](int, int i, int j) {
    T s = 0;
#pragma unroll
    for (int k = 0; k < L0; ++k) s += S0[k * P0 + i] * A[j * P0 + k];
    B[j * P0 + i] = s;
  });
  __syncthreads();
  each([&](int, int i, int j) {
    T s = 0;
#pragma unroll
    for (int k = 0; k < L1; ++k) s += S1[k * P1 + j] * B[k * P0 + i];
    A[j * P0 + i] = div_nr(s, sl[i] + sl[L0 + j]);
  });
  __syncthreads();
  each([&](int, int i, int j) {
    T s = 0;
#pragma unroll
    for (int k = 0; k < L1; ++k) s += S1[j * P1 + k] * A[k * P0 + i];
    B[j * P0 + i] = s;
  });
  __syncthreads();
  auto* out = (__attribute__((address_space(1))) T*)po + (int64_t)pid * N;
  each([&](int, int i, int j) {
    T s = 0;
#pragma unroll
    for (int k = 0; k < L0; ++k) s += S0[i * P0 + k] * B[j * P0 + k];
    out[j * L0 + i] = (sw[i] * sw[L0 + j]) * s;
  });
}
// The form of a grid's 2D sweep (patches: of the grid, also when grids share a launch, so
// that a batch gives what its grids give alone).
template <class T>
bool fdm2_fits(int NA, int NL, int patches) {
  return NA * NL <= FDM2_NODES && (int64_t)patches * NA * NL * (int64_t)sizeof(T) <= FDM2_BYTES;
}

template <class T, int NA, int NL, bool BATCH>
int fdm2_go(int nd, const FdmArgs<T>& a, const BatchList<FdmArgs<T>>& bl, int nlog, hipStream_t s) {
  const auto go = [&](auto kernel, int th) { hipLaunchKernelGGL(kernel, dim3(xcd_grid(nlog)), dim3(th), 0, s, a, bl, nlog); };
  if (nd == 0) go(fdm2_kernel<T, NA, NL, 0, BATCH>, fdm2_threads<NA, NL, 0>());
  else if (nd == 1) go(fdm2_kernel<T, NA, NL, 1, BATCH>, fdm2_threads<NA, NL, 1>());
  else if constexpr (NA == NL) go(fdm2_kernel<T, NA, NL, -1, BATCH>, fdm2_threads<NA, NL, -1>());
  else return -4;
  return 0;
}

// waves: wavefronts per block (1 .. 8; 0 = default), the shape the autotuner picks.
template <class T, int DIM, int NA, int NL, bool BATCH>
int fdm_go(int nd, const FdmArgs<T>& a, const BatchList<FdmArgs<T>>& bl, int nlog, int waves, hipStream_t s) {
  constexpr size_t shm = fdm_shmem<T, NA, NL, DIM>();
  const int th = (waves >= 1 && waves <= 8) ? 64 * waves : fdm_threads<NA, NL, DIM>();
  if (nd < 0) {
    if constexpr (NA == NL) {
      fdm_launch_nd<T, DIM, NA, NL, -1, BATCH>(a, bl, nlog, th, shm, s);
      return 0;
    }
    return -4;
  }
  if (nd == 0) fdm_launch_nd<T, DIM, NA, NL, 0, BATCH>(a, bl, nlog, th, shm, s);
  else if (nd == 1) fdm_launch_nd<T, DIM, NA, NL, 1, BATCH>(a, bl, nlog, th, shm, s);
  else if constexpr (DIM == 3) fdm_launch_nd<T, DIM, NA, NL, 2, BATCH>(a, bl, nlog, th, shm, s);
  else return -4;
  return 0;
}

// ================================================================ multiplicative update
// u += R_s^T Delta u_s, unweighted, for the patches of one launch of the patch
// solve (a colour class: their node sets are disjoint, so every node receives
// at most one value and no two threads write the same entry).  One block per
// patch (its index among the launch's patches, as the patch solve numbered
// them), threads over its tile in grid-natural order; positions outside a
// Dirichlet domain are skipped.
template <class T, int DIM>
__global__ void __launch_bounds__(256) mult_update_kernel(LevelDev<T> L, int nd, int NA, int NL, PatchLat lat,
                                                          int npx, int npy, int swp, const T* __restrict__ buf,
                                                          T* __restrict__ u) {
  if (inactive(L.active)) return;
  const int pid = blockIdx.x;
  int p[3];
  p[0] = lat.start[0] + lat.stride[0] * (pid % npx);
  p[1] = lat.start[1] + lat.stride[1] * ((pid / npx) % npy);
  p[2] = DIM == 3 ? lat.start[2] + lat.stride[2] * (pid / (npx * npy)) : 0;
  const int* go[3] = {nullptr, nullptr, nullptr};
  int len[3] = {1, 1, 1};
  for (int d = 0; d < DIM; ++d) {
    const bool fc = d == nd;
    len[d] = fc ? NA : NL;
    go[d] = fc ? L.dir[d].goff_fc + p[d] * NA : L.dir[d].goff_ec + p[d] * NL;
  }
  const int ts = len[0] * len[1] * len[2];
  const T* src = buf + (int64_t)pid * ts;
  for (int q = threadIdx.x; q < ts; q += blockDim.x) {
    const int o0 = q % len[0], rw = q / len[0];
    const int o1 = swp ? rw / len[2] : rw % len[1], o2 = swp ? rw % len[2] : rw / len[1];
    const int g0 = go[0][o0], g1 = go[1][o1], g2 = DIM == 3 ? go[2][o2] : 0;
    if ((g0 | g1 | g2) < 0) continue;
    u[g0 + g1 + g2] += src[q];
  }
}

template <class T, int DIM>
int mult_update_launch(const LevelDev<T>& L, int nd, int NA, int NL, const PatchLat& lat, int npx, int npy,
                       int npz, int swp, const T* buf, T* u, hipStream_t s) {
  const int npatch = npx * npy * (DIM == 3 ? npz : 1);
  if (npatch <= 0) return 0;
  hipLaunchKernelGGL((mult_update_kernel<T, DIM>), dim3(npatch), dim3(256), 0, s, L, nd, NA, NL, lat, npx, npy, swp,
                     buf, u);
  return 0;
}

// ================================================================ overlap summation
// u += sum_s R_s^T (w_s Delta u_s) (assign: u = the sum, for u = 0 on entry),
// gathered per node in a fixed order over the
// (at most 2 x 3 x 3) covering patches: deterministic, no atomics.  One block
// per group of elements; per element and direction the candidate patches of
// each local index are tabulated in LDS as address components, so a node's sum
// is a few loads at addresses Ax[i] + Ay[j] + Az[k].
template <int NP, int DIM>
constexpr int combine_epb() {
  return imax(1, 256 / ipow(NP, DIM));
}
// Large elements are split over several blocks of at most COMBINE_CHUNK nodes
// (a whole P = 32 element per block left 512 blocks, each thread looping 140
// times through latency-bound candidate loads).
constexpr int COMBINE_CHUNK = 2048;
template <int NP, int DIM>
constexpr int combine_bpe() {
  return combine_epb<NP, DIM>() == 1 ? (ipow(NP, DIM) + COMBINE_CHUNK - 1) / COMBINE_CHUNK : 1;
}

template <class T>
struct CombArgs {
  LevelDev<T> L;
  const T* buf = nullptr;  // the patch solve's weighted corrections
  T* u = nullptr;
  int nd = -1, NA = 0, NL = 0;
  int npx = 1, npy = 1, npz = 1;
  PatchBuf pb;
  int nblk = 0;
  int assign = 0;
};

// BATCH: the arguments come from the work list bl (ntot logical blocks in all)
template <class T, int DIM, int NP, int MAXC, bool BATCH = false>
__global__ void __launch_bounds__(256) combine_kernel(CombArgs<T> a0, BatchList<CombArgs<T>> bl, int ntot) {
  constexpr int NE = ipow(NP, DIM), EPB = combine_epb<NP, DIM>(), BPE = combine_bpe<NP, DIM>();
  constexpr int P = NP - 1;
  constexpr int CZ = DIM == 3 ? MAXC : 1;
  __shared__ int64_t cadr[EPB][3][NP][MAXC];
  __shared__ int ccnt[EPB][3][NP];
  __shared__ __align__(16) int sargs_raw[BATCH ? sizeof(CombArgs<T>) / sizeof(int) : 1];
  CombArgs<T>* sargs = reinterpret_cast<CombArgs<T>*>(sargs_raw);
  const CombArgs<T>* ap;
  int blk;
  if constexpr (BATCH) {
    const int b = xcd_block(ntot);
    if (b < 0) return;
    blk = batch_pick(bl, b, sargs);
    ap = sargs;
  } else {
    blk = xcd_block(a0.nblk);
    if (blk < 0) return;
    ap = &a0;
  }
  const LevelDev<T>& L = ap->L;
  const T* __restrict__ buf = ap->buf;
  T* __restrict__ u = ap->u;
  const int nd = ap->nd, NA = ap->NA, NL = ap->NL, npx = ap->npx, npy = ap->npy;
  const bool assign = ap->assign != 0;
  if (inactive(L.active)) return;
  // BPE > 1: block blk takes nodes [q_lo, q_hi) of element blk / BPE
  const int e0 = BPE > 1 ? blk / BPE : blk * EPB;
  const int ne = BPE > 1 ? 1 : imin(EPB, L.n_elem - e0);
  const int q_lo = BPE > 1 ? (blk % BPE) * COMBINE_CHUNK : 0;
  const int q_hi = BPE > 1 ? imin(NE, q_lo + COMBINE_CHUNK) : ne * NE;
  const int tid = threadIdx.x, nth = blockDim.x;
  const int N1 = L.dir[0].N, N2 = L.dir[1].N, NO = L.NO;
  int len[3] = {1, 1, 1};
  for (int d = 0; d < DIM; ++d) len[d] = (d == nd) ? NA : NL;
  const int K = ap->pb.K, step = ap->pb.step, swp = ap->pb.swp;
  const int nsy = (npy + K - 1) / K;
  const int64_t TS = (int64_t)len[0] * ((K - 1) * step + len[1]) * len[2];
  const int64_t pst[3] = {1, npx, (int64_t)npx * nsy};
  const int64_t ost[3] = {1, swp ? (int64_t)len[0] * len[2] : len[0], swp ? len[0] : (int64_t)len[0] * len[1]};
  for (int q = tid; q < ne * DIM * NP; q += nth) {
    const int el = q / (DIM * NP), rem = q - el * DIM * NP, d = rem / NP, i = rem - d * NP;
    const int e = e0 + el;
    const int md = d == 0 ? e % N1 : (d == 1 ? (DIM == 3 ? (e / N1) % N2 : e / N1) : e / (N1 * N2));
    const DirDev<T>& dd = L.dir[d];
    const int N = dd.N;
    int c = 0;
    int cp[3], co[3];
    if (d == nd) {  // faces m (tile position P + i, needs i < P) and m + 1 (position i - 1, needs i >= 1)
      if (i < P) { cp[c] = md; co[c++] = P + i; }
      if (i >= 1) { cp[c] = dd.periodic ? (md + 1) % N : md + 1; co[c++] = i - 1; }
    } else {        // element-centred patches m - 1, m, m + 1
      if (i < NO && (dd.periodic || md > 0)) { cp[c] = (md - 1 + N) % N; co[c++] = NP + NO + i; }
      cp[c] = md; co[c++] = i + NO;
      if (i >= NP - NO && (dd.periodic || md < N - 1)) { cp[c] = (md + 1) % N; co[c++] = i - NP + NO; }
    }
    if (d == 1 && K > 1) {  // strips: patches of one strip meet in one plane of its summed tile
      int n = 0;
      for (int k = 0; k < c; ++k) {
        const int st = cp[k] >> __builtin_ctz(K), pl = (cp[k] & (K - 1)) * step + co[k];
        bool same = false;
        for (int j = 0; j < n; ++j) same = same || (cp[j] == st && co[j] == pl);
        if (!same) { cp[n] = st; co[n++] = pl; }
      }
      c = n;
    }
    ccnt[el][d][i] = c;
    for (int k = 0; k < MAXC; ++k) cadr[el][d][i][k] = k < c ? cp[k] * pst[d] * TS + co[k] * ost[d] : 0;
  }
  if (DIM == 2)
    for (int q = tid; q < ne; q += nth) {
      ccnt[q][2][0] = 1;
      for (int k = 0; k < MAXC; ++k) cadr[q][2][0][k] = 0;
    }
  __syncthreads();
  // each node: all its (at most MAXC per direction) candidates are loaded before
  // the sum, then added in a fixed order (z, y, x candidates)
  const int64_t g0 = (int64_t)e0 * NE;
  for (int q = q_lo + tid; q < q_hi; q += nth) {
    const int el = q / NE, loc = q - el * NE;
    const int i = loc % NP, j = (loc / NP) % NP, k = DIM == 3 ? loc / (NP * NP) : 0;
    const int nx = ccnt[el][0][i], ny = ccnt[el][1][j], nz = ccnt[el][2][k];
    T v[CZ][MAXC][MAXC];
#pragma unroll
    for (int c = 0; c < CZ; ++c)
#pragma unroll
      for (int b = 0; b < MAXC; ++b)
#pragma unroll
        for (int a = 0; a < MAXC; ++a) {
          // invalid candidates are not loaded (their lanes are masked off: on
          // average about half of the 2 x 2 x 2 slots are empty) and add 0
          const bool ok = c < nz && b < ny && a < nx;
          T val = T(0);
          if (ok) val = buf[cadr[el][2][k][c] + cadr[el][1][j][b] + cadr[el][0][i][a]];
          v[c][b][a] = val;
        }
    T s = 0;
#pragma unroll
    for (int c = 0; c < CZ; ++c)
#pragma unroll
      for (int b = 0; b < MAXC; ++b)
#pragma unroll
        for (int a = 0; a < MAXC; ++a)
          s += T(c < nz && b < ny && a < nx ? 1 : 0) * v[c][b][a];  // s + 0 v = s: order unchanged
    if (assign)
      u[g0 + q] = s;
    else
      u[g0 + q] += s;
  }
}

// Blocks of one grid's overlap summation.
template <int DIM, int NP>
int combine_blocks(int n_elem) {
  constexpr int EPB = combine_epb<NP, DIM>(), BPE = combine_bpe<NP, DIM>();
  return BPE > 1 ? n_elem * BPE : (n_elem + EPB - 1) / EPB;
}
// 3D, at most two covering patches per direction: a thread owns a line of nodes along one
// direction C (1 or 2) of one element; the lanes run over directions 0 and B = 3 - C of a
// layer of elements (equal index in direction C), whole blocks of lines.  What a node
// needs in directions 0 and B (32-bit offsets, which candidates exist) is then worked out
// once per line, and the covering patches in direction C are the same for the whole block:
// their addresses are scalars, and where there is one no load is issued for a second.
// C is the slower direction of the tiles, so that a wave's loads run through consecutive
// rows; with the other choice a load took 45 cache accesses and the address unit bound the
// kernel (32^3 P = 8 FP32: 165 us, now 133 us or 3.5 TB/s; 150 us for a thread per node with
// table reads from LDS.  32^3 P = 4: 37 -> 24 us, 9x7x11 P = 12: 16 -> 11 us; FP64 16^3 P = 8
// 24 us, 5.3 TB/s, either way).
// Existing candidates are added in the same order either way (directions 2, 1, 0).
template <class T>
struct Comb3Args {
  const T* buf = nullptr;
  T* u = nullptr;
  const int* active = nullptr;
  int64_t psc = 0;  // elements from patch to patch along C
  int c1 = 0;       // C is direction 1
  int N0 = 1, NB = 1, NC = 1, per = 0, NO = 0, nd = -1;  // (per: bit 0 direction 0, 1 B, 2 C; nd: 0, 1 = B, 2 = C)
  int ts = 0, psb = 0, ostb = 0, ostc = 0;               // tile; patches along B; positions of a tile
  int K = 1, step = 0;
  int eb = 0, ec = 0;                                    // element strides of the level vector along B and C
  int nline = 0, bpl = 1, nblk = 0, assign = 0;          // lines and blocks of a layer
  uint32_t mg0 = 0, mgb = 0;                             // divisions by N0 and bpl
};
constexpr int COMB3_THREADS = 256;

template <class T>
Comb3Args<T> combine3_args(const LevelDev<T>& L, int nd, int NA, int NL, const T* buf, T* u, int npx, int npy, int npz,
                           const PatchBuf& pb, bool assign) {
  Comb3Args<T> a;
  const int l0 = nd == 0 ? NA : NL, l1 = nd == 1 ? NA : NL, l2 = nd == 2 ? NA : NL;
  const int nsy = (npy + pb.K - 1) / pb.K;
  const int64_t ps1 = (int64_t)l0 * ((pb.K - 1) * pb.step + l1) * l2 * npx, ps2 = ps1 * nsy;
  const int ost1 = pb.swp ? l0 * l2 : l0, ost2 = pb.swp ? l0 : l0 * l1;
  const int N1 = L.dir[1].N, N2 = L.dir[2].N;
  const bool c1 = pb.swp && ps2 * npz * (int64_t)sizeof(T) < (int64_t(1) << 32) && ps2 * npz < (int64_t(1) << 31);
  a.buf = buf;
  a.u = u;
  a.active = L.active;
  a.c1 = c1 ? 1 : 0;
  a.ts = (int)(ps1 / npx);
  a.psc = c1 ? ps1 : ps2;
  a.psb = (int)(c1 ? ps2 : ps1);
  a.ostb = c1 ? ost2 : ost1;
  a.ostc = c1 ? ost1 : ost2;
  a.N0 = L.dir[0].N;
  a.NB = c1 ? N2 : N1;
  a.NC = c1 ? N1 : N2;
  a.eb = c1 ? a.N0 * N1 : a.N0;
  a.ec = c1 ? a.N0 : a.N0 * N1;
  const int B = c1 ? 2 : 1, C = 3 - B;
  a.per = (L.dir[0].periodic ? 1 : 0) | (L.dir[B].periodic ? 2 : 0) | (L.dir[C].periodic ? 4 : 0);
  a.NO = L.NO;
  a.nd = nd <= 0 ? nd : (nd == B ? 1 : 2);
  a.K = pb.K;
  a.step = pb.step;
  a.nline = a.N0 * a.NB * L.NP * L.NP;
  a.bpl = (a.nline + COMB3_THREADS - 1) / COMB3_THREADS;
  a.nblk = a.bpl * a.NC;
  a.assign = assign ? 1 : 0;
  a.mg0 = div_magic((int64_t)a.N0 * a.NB, a.N0);
  a.mgb = div_magic(a.nblk, a.bpl);
  return a;
}
// Candidate slots per node and direction: three covering element-centred
// patches in one direction only when 2 N_O > N_P.
inline int combine_maxc(int NP, int NO) { return 2 * NO > NP ? 3 : 2; }
// The offsets inside a layer of patches have to fit 32 bits (bytes), the lines an int; larger
// grids and three candidates take combine_kernel.
template <class T>
bool combine3_fits(int dim, int NP, int NO, int nd, int NA, int NL, const int* N, int npx, int npy, const PatchBuf& pb) {
  if (dim != 3 || combine_maxc(NP, NO) != 2) return false;
  const int64_t l0 = nd == 0 ? NA : NL, l1 = nd == 1 ? NA : NL, l2 = nd == 2 ? NA : NL;
  const int64_t layer = l0 * ((pb.K - 1) * (int64_t)pb.step + l1) * l2 * npx * ((npy + pb.K - 1) / pb.K);
  const int64_t lines = (int64_t)N[0] * N[1] * N[2] * NP * NP;
  return layer < (int64_t(1) << 31) && layer * (int64_t)sizeof(T) < (int64_t(1) << 32) && lines < (int64_t(1) << 31);
}

// BATCH: the arguments come from the work list bl (ntot logical blocks in all)
template <class T, int NP, bool BATCH = false>
__global__ void __launch_bounds__(COMB3_THREADS)
    combine3_kernel(Comb3Args<T> a0, BatchList<Comb3Args<T>> bl, int ntot) {
  constexpr int NLN = NP * NP, P = NP - 1;
  constexpr int KC = imin(NP, 3);  // nodes of a line whose loads are issued together
  __shared__ __align__(16) int sargs_raw[BATCH ? sizeof(Comb3Args<T>) / sizeof(int) : 1];
  const Comb3Args<T>* ap;
  int blk = 0;
  if constexpr (BATCH) {
    const int b = xcd_block(ntot);
    if (b < 0) return;
    Comb3Args<T>* sargs = reinterpret_cast<Comb3Args<T>*>(sargs_raw);
    blk = batch_pick(bl, b, sargs);
    ap = sargs;
  } else {
    ap = &a0;
  }
  // every argument into scalar registers by one group of loads
  const auto uni = [](int v) { return BATCH ? __builtin_amdgcn_readfirstlane(v) : v; };
  const auto ptr = [](auto* q) { return BATCH ? sgpr_ptr(q) : q; };
  const T* pbuf = ptr(ap->buf);
  T* pu = ptr(ap->u);
  const int* act = ptr(ap->active);
  int64_t psc = ap->psc;
  if constexpr (BATCH) psc = (int64_t)(uint32_t)uni((int)psc) | ((int64_t)uni((int)(psc >> 32)) << 32);
  int N0 = uni(ap->N0), NB = uni(ap->NB), NC = uni(ap->NC), per = uni(ap->per), NO = uni(ap->NO), nd = uni(ap->nd);
  int ts = uni(ap->ts), psb = uni(ap->psb), ostb = uni(ap->ostb), ostc = uni(ap->ostc), K = uni(ap->K);
  int step = uni(ap->step), eb = uni(ap->eb), ec = uni(ap->ec), c1 = uni(ap->c1);
  int nline = uni(ap->nline), bpl = uni(ap->bpl), nblk = uni(ap->nblk), assign = uni(ap->assign);
  uint32_t mg0 = uni(ap->mg0), mgb = uni(ap->mgb);
  if constexpr (!BATCH) {
    asm volatile("" : "+s"(pbuf), "+s"(pu), "+s"(act), "+s"(psc), "+s"(N0), "+s"(NB), "+s"(NC), "+s"(per), "+s"(NO),
                 "+s"(nd), "+s"(ts), "+s"(psb), "+s"(ostb), "+s"(ostc));
    asm volatile("" : "+s"(K), "+s"(step), "+s"(eb), "+s"(ec), "+s"(c1), "+s"(nline), "+s"(bpl), "+s"(nblk),
                 "+s"(assign), "+s"(mg0), "+s"(mgb));
    blk = xcd_block(nblk);
    if (blk < 0) return;
  }
  using G = const __attribute__((address_space(1))) T;  // global memory
  using GC = const __attribute__((address_space(1))) char;
  if (act != nullptr && *(const __attribute__((address_space(1))) int*)act == 0) return;
  blk = uni(blk);
  const int mc = uni(div_by(blk, bpl, mgb));
  const int ln = (blk - mc * bpl) * COMB3_THREADS + (int)threadIdx.x;
  if (ln >= nline) return;
  const int el = ln / NLN, t = ln - el * NLN, i = t % NP, j = t / NP;
  const int mb = div_by(el, N0, mg0), m0 = el - mb * N0;
  // covering patches of index i of element m: (p, o) and, if two, (p2, o2), in order
  const auto cover = [&](int m, int N, bool wrap, bool face, int i, int& p, int& o, int& p2, int& o2) {
    bool two;
    if (face) {  // faces m (position P + i, i < P) and m + 1 (position i - 1, i >= 1)
      const int q = wrap && m + 1 == N ? 0 : m + 1;
      two = i >= 1 && i < P;
      p = i < P ? m : q;
      o = i < P ? P + i : i - 1;
      p2 = q;
      o2 = i - 1;
    } else {  // element-centred patches m - 1, m, m + 1
      const bool lo = i < NO && (wrap || m > 0), hi = i >= NP - NO && (wrap || m < N - 1);
      two = lo || hi;
      p = lo ? (m > 0 ? m - 1 : N - 1) : m;
      o = lo ? NP + NO + i : i + NO;
      p2 = lo ? m : (m < N - 1 ? m + 1 : 0);
      o2 = lo ? i + NO : i - NP + NO;
    }
    return two;
  };
  const int sh = __builtin_ctz(K);
  // strips (along direction 1): patches of one strip meet in one plane of its summed tile
  const auto strip = [&](bool two, int& p, int& o, int& p2, int& o2) {
    o += (p & (K - 1)) * step;
    o2 += (p2 & (K - 1)) * step;
    p >>= sh;
    p2 >>= sh;
    return two && !(p == p2 && o == o2);
  };
  int pa, oa, pb, ob;
  const bool x2 = cover(m0, N0, per & 1, nd == 0, i, pa, oa, pb, ob);
  const uint32_t ax = (uint32_t)(pa * ts + oa) * (uint32_t)sizeof(T), bx = (uint32_t)(pb * ts + ob) * (uint32_t)sizeof(T);
  bool b2 = cover(mb, NB, per & 2, nd == 1, j, pa, oa, pb, ob);
  if (!c1) b2 = strip(b2, pa, oa, pb, ob);
  const uint32_t ab = (uint32_t)(pa * psb + oa * ostb) * (uint32_t)sizeof(T);
  const uint32_t bb = (uint32_t)(pb * psb + ob * ostb) * (uint32_t)sizeof(T);
  const bool xb = x2 && b2;
  const int ub = c1 ? NP * NP : NP, uc = c1 ? NP : NP * NP;
  auto* u = (__attribute__((address_space(1))) T*)pu + ((int64_t)m0 + (int64_t)mb * eb + (int64_t)mc * ec) * (NP * NLN) +
            (i + j * ub);
#pragma unroll
  for (int k0 = 0; k0 < NP; k0 += KC) {
    constexpr int LAST = (NP - 1) / KC * KC;
    const int kn = k0 == LAST ? NP - LAST : KC;
    T v[KC][2][4], old[KC];
    bool two[KC], any = false;
    int64_t z[KC][2];
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      if (c >= kn) continue;
      int p, o, p2, o2;
      two[c] = cover(mc, NC, per & 4, nd == 2, k0 + c, p, o, p2, o2);
      if (c1) two[c] = strip(two[c], p, o, p2, o2);
      any = any || two[c];
      z[c][0] = p * psc + (int64_t)o * ostc;
      z[c][1] = two[c] ? p2 * psc + (int64_t)o2 * ostc : z[c][0];  // (repeated and unused where there is one)
    }
    const auto load = [&](int h, int q, uint32_t off) {
#pragma unroll
      for (int c = 0; c < KC; ++c)
        if (c < kn) v[c][h][q] = *(G*)((GC*)((G*)pbuf + z[c][h]) + off);
    };
#pragma unroll
    for (int c = 0; c < KC; ++c)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int q = 0; q < 4; ++q) v[c][h][q] = T(0);
#pragma unroll
    for (int c = 0; c < KC; ++c)
      if (c < kn) old[c] = assign ? T(0) : u[(k0 + c) * uc];
    load(0, 0, ab + ax);
    if (any) load(1, 0, ab + ax);
    if (x2) {
      load(0, 1, ab + bx);
      if (any) load(1, 1, ab + bx);
    }
    if (b2) {
      load(0, 2, bb + ax);
      if (any) load(1, 2, bb + ax);
    }
    if (xb) {
      load(0, 3, bb + bx);
      if (any) load(1, 3, bb + bx);
    }
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      if (c >= kn) continue;
      T s;
      // (absent candidates are 0 and change nothing)
      if (c1) {  // C = 1: directions 2 (B), 1 (C), 0
        s = v[c][0][0] + v[c][0][1];
        if (two[c]) s = (s + v[c][1][0]) + v[c][1][1];
        s = (s + v[c][0][2]) + v[c][0][3];
        if (two[c]) s = (s + v[c][1][2]) + v[c][1][3];
      } else {   // C = 2: directions 2 (C), 1 (B), 0
        s = ((v[c][0][0] + v[c][0][1]) + v[c][0][2]) + v[c][0][3];
        if (two[c]) s = (((s + v[c][1][0]) + v[c][1][1]) + v[c][1][2]) + v[c][1][3];
      }
      u[(k0 + c) * uc] = assign ? s : old[c] + s;
    }
  }
}

template <class T, int NP>
int combine3_launch(const Comb3Args<T>& a, hipStream_t s) {
  hipLaunchKernelGGL((combine3_kernel<T, NP, false>), dim3(xcd_grid(a.nblk)), dim3(COMB3_THREADS), 0, s, a,
                     BatchList<Comb3Args<T>>{}, a.nblk);
  return 0;
}
// One launch over the overlap summations of many grids (ntot logical blocks in all).
template <class T, int NP>
int combine3_batch_launch(const BatchList<Comb3Args<T>>& bl, int ntot, hipStream_t s) {
  hipLaunchKernelGGL((combine3_kernel<T, NP, true>), dim3(xcd_grid(ntot)), dim3(COMB3_THREADS), 0, s, Comb3Args<T>{}, bl,
                     ntot);
  return 0;
}

template <class T, int DIM, int NP>
int combine_launch_t(const LevelDev<T>& L, int nd, int NA, int NL, const T* buf, T* u, int npx,
                     int npy, int npz, const PatchBuf& pb, bool assign, hipStream_t s) {
  if constexpr (DIM == 3) {
    const int N[3] = {L.dir[0].N, L.dir[1].N, L.dir[2].N};
    if (combine3_fits<T>(3, NP, L.NO, nd, NA, NL, N, npx, npy, pb))
      return combine3_launch<T, NP>(combine3_args(L, nd, NA, NL, buf, u, npx, npy, npz, pb, assign), s);
  }
  CombArgs<T> a;
  a.L = L;
  a.buf = buf;
  a.u = u;
  a.nd = nd;
  a.NA = NA;
  a.NL = NL;
  a.npx = npx;
  a.npy = npy;
  a.npz = npz;
  a.pb = pb;
  a.nblk = combine_blocks<DIM, NP>(L.n_elem);
  a.assign = assign ? 1 : 0;
  if (combine_maxc(NP, L.NO) == 3)
    hipLaunchKernelGGL((combine_kernel<T, DIM, NP, 3, false>), dim3(xcd_grid(a.nblk)), dim3(256), 0, s, a,
                       BatchList<CombArgs<T>>{}, a.nblk);
  else
    hipLaunchKernelGGL((combine_kernel<T, DIM, NP, 2, false>), dim3(xcd_grid(a.nblk)), dim3(256), 0, s, a,
                       BatchList<CombArgs<T>>{}, a.nblk);
  return 0;
}

// One launch over the overlap summations of many grids (same NP and candidate
// slots maxc): ntot logical blocks, grid g's combine_blocks in the range of bl.
template <class T, int DIM, int NP>
int combine_batch_launch(int maxc, const BatchList<CombArgs<T>>& bl, const BatchList<Comb3Args<T>>& bl3, int ntot,
                         hipStream_t s) {
  if constexpr (DIM == 3)
    if (maxc == 0) return combine3_batch_launch<T, NP>(bl3, ntot, s);  // grids that combine3_fits
  if (maxc == 3)
    hipLaunchKernelGGL((combine_kernel<T, DIM, NP, 3, true>), dim3(xcd_grid(ntot)), dim3(256), 0, s, CombArgs<T>{},
                       bl, ntot);
  else
    hipLaunchKernelGGL((combine_kernel<T, DIM, NP, 2, true>), dim3(xcd_grid(ntot)), dim3(256), 0, s, CombArgs<T>{},
                       bl, ntot);
  return 0;
}

// ================================================================ p-transfers
// Element-local tensor-product contractions with the embedded interpolation J
// (NPf x NPc).  RESTRICT: out_c = (J^T x J^T x J^T) in_f.  Otherwise:
// out_f += (J x J x J) in_c.  One block per group of elements; LDS ping-pong.
constexpr int XFER_THREADS = 256;  // block size of transfer_kernel (its copies unroll over it)
template <int NPF, int DIM>
constexpr int xfer_epb() {
  return imax(1, 512 / ipow(NPF, DIM));
}

// One contraction pass of the transfer along direction D, all extents known at
// compile time: before the pass directions < D have NOUT points and the others
// NIN; the pass maps direction D from NIN to NOUT points.
template <class T, int DIM, int NIN, int NOUT, int NEF, int D, bool RESTRICT, int NPC>
__device__ __forceinline__ void xfer_pass(const T* __restrict__ sJ, const T* __restrict__ src,
                                          T* __restrict__ dst, int ne) {
  constexpr int n0 = D > 0 ? NOUT : NIN, n1 = D > 1 ? NOUT : NIN;
  constexpr int m0 = NOUT * (D == 0) + n0 * (D != 0);
  constexpr int m1 = DIM >= 2 ? (D >= 1 ? NOUT : NIN) : 1;
  constexpr int m2 = DIM == 3 ? (D == 2 ? NOUT : NIN) : 1;
  constexpr int per = m0 * m1 * m2;
  constexpr int SK = D == 0 ? 1 : (D == 1 ? n0 : n0 * n1);  // source stride of direction D
  for (int q = threadIdx.x; q < ne * per; q += blockDim.x) {
    const int el = q / per, r = q - el * per;
    const int i0 = r % m0, i1 = (r / m0) % m1, i2 = r / (m0 * m1);
    const int iout = D == 0 ? i0 : (D == 1 ? i1 : i2);
    // source position with the direction-D index set to 0
    const int j0 = D == 0 ? 0 : i0, j1 = D == 1 ? 0 : i1, j2 = D == 2 ? 0 : i2;
    const T* sp = src + el * NEF + (j2 * n1 + j1) * n0 + j0;
    T s = 0;
#pragma unroll
    for (int k = 0; k < NIN; ++k) {
      const T jv = RESTRICT ? sJ[k * NPC + iout] : sJ[iout * NPC + k];
      s += jv * sp[k * SK];
    }
    dst[el * NEF + r] = s;
  }
}

template <class T>
struct XferArgs {
  const T* J = nullptr;
  int n_elem = 0;
  const T* in = nullptr;
  T* out = nullptr;
  const int* active = nullptr;
};

// BATCH: the arguments come from the work list bl (ntot logical blocks in all)
template <class T, int DIM, int NPF, int NPC, bool RESTRICT, bool BATCH = false>
__global__ void __launch_bounds__(512) transfer_kernel(XferArgs<T> a0, BatchList<XferArgs<T>> bl, int ntot) {
  __shared__ __align__(16) int sargs_raw[BATCH ? sizeof(XferArgs<T>) / sizeof(int) : 1];
  XferArgs<T>* sargs = reinterpret_cast<XferArgs<T>*>(sargs_raw);
  const XferArgs<T>* ap;
  int blk = blockIdx.x;
  if constexpr (BATCH) {
    const int b = xcd_block(ntot);
    if (b < 0) return;
    blk = batch_pick(bl, b, sargs);
    ap = sargs;
  } else {
    ap = &a0;
  }
  const T* __restrict__ J = ap->J;
  const int n_elem = ap->n_elem;
  const T* __restrict__ in = ap->in;
  T* __restrict__ out = ap->out;
  if (inactive(ap->active)) return;
  constexpr int NEF = ipow(NPF, DIM), EPB = xfer_epb<NPF, DIM>();
  constexpr int NIN = RESTRICT ? NPF : NPC, NOUT = RESTRICT ? NPC : NPF;
  constexpr int NEI = ipow(NIN, DIM), NEO = ipow(NOUT, DIM);
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* bufA = reinterpret_cast<T*>(smem_raw);
  T* bufB = bufA + EPB * NEF;
  __shared__ T sJ[NPF * NPC];
  const int e0 = blk * EPB;
  const int ne = imin(EPB, n_elem - e0);
  staged_copy<T, XFER_THREADS, NPF * NPC>([&](int q) { return J[q]; }, [&](int q, T v) { sJ[q] = v; });
  staged_copy<T, XFER_THREADS, EPB * NEI>([&](int q) { return in[(int64_t)e0 * NEI + q]; },
                                          [&](int q, T v) {
                                            const int el = q / NEI;
                                            bufA[el * NEF + q - el * NEI] = v;  // per-element stride NEF in LDS
                                          },
                                          ne * NEI);
  __syncthreads();
  xfer_pass<T, DIM, NIN, NOUT, NEF, 0, RESTRICT, NPC>(sJ, bufA, bufB, ne);
  __syncthreads();
  xfer_pass<T, DIM, NIN, NOUT, NEF, 1, RESTRICT, NPC>(sJ, bufB, bufA, ne);
  __syncthreads();
  const T* res = bufA;
  if constexpr (DIM == 3) {
    xfer_pass<T, DIM, NIN, NOUT, NEF, 2, RESTRICT, NPC>(sJ, bufA, bufB, ne);
    __syncthreads();
    res = bufB;
  }
  const auto rv = [&](int q) {
    const int el = q / NEO;
    return res[el * NEF + q - el * NEO];
  };
  T* o = out + (int64_t)e0 * NEO;
  if constexpr (RESTRICT)
    staged_copy<T, XFER_THREADS, EPB * NEO>(rv, [&](int q, T v) { o[q] = v; }, ne * NEO);
  else
    staged_copy<T, XFER_THREADS, EPB * NEO>([&](int q) { return o[q]; }, [&](int q, T v) { o[q] = v + rv(q); },
                                            ne * NEO);
}

// 3D at orders from 12 on, an element per block: a thread contracts whole lines, values in
// registers and J in scalar registers, where transfer_kernel reads both operands of every
// product from LDS.  Direction 2, whose lines' lanes run along the vector, is contracted
// first by the restriction, from global memory, and last by the prolongation, into it.
// 7x9x6 P = 16 FP64 (32 MB): restriction 14.6 -> 8.4 us, prolongation 18.5 -> 8.5 us;
// 9x7x11 P = 12 FP32: 5.6 -> 3.1 and 6.9 -> 4.1 us.  12 is where it has been brought in, not
// where it ends: timed in its place at lower orders it is the faster form there too
// (transfer_kernel / this, restriction and prolongation, us: 32^3 P = 8 FP64 67 / 32 and 75 / 63,
// FP32 42 / 18 and 51 / 34; 32^3 P = 4 FP64 13.6 / 9.7 and 16.4 / 14.8; 8^3 P = 8 3.7 / 3.6).
template <int NPF>
constexpr bool xfer_lines() {
  return NPF >= 12;
}
template <class T, int NPF, int NPC, bool RESTRICT, bool BATCH = false>
__global__ void __launch_bounds__((round64(NPF * NPF)))
    transfer3_kernel(XferArgs<T> a0, BatchList<XferArgs<T>> bl, int ntot) {
  constexpr int TH = round64(NPF * NPF), NF = NPF * NPF * NPF, NC = NPC * NPC * NPC;
  __shared__ T A[NPF * NPF * NPC], B[NPF * NPC * NPC];
  __shared__ __align__(16) int sargs_raw[BATCH ? sizeof(XferArgs<T>) / sizeof(int) : 1];
  const XferArgs<T>* ap;
  int blk = 0;
  if constexpr (BATCH) {
    const int b = xcd_block(ntot);
    if (b < 0) return;
    XferArgs<T>* sargs = reinterpret_cast<XferArgs<T>*>(sargs_raw);
    blk = batch_pick(bl, b, sargs);
    ap = sargs;
  } else {
    ap = &a0;
    blk = blockIdx.x;
  }
  const auto ptr = [](auto* q) { return BATCH ? sgpr_ptr(q) : q; };
  if (inactive(ptr(ap->active))) return;
  using G = const __attribute__((address_space(1))) T;   // global memory
  using CT = const __attribute__((address_space(4))) T;  // constant: scalar loads
  CT* J = (CT*)ptr(ap->J);
  blk = __builtin_amdgcn_readfirstlane(blk);
  const int tid = threadIdx.x;
  if constexpr (RESTRICT) {
    G* in = (G*)ptr(ap->in) + (int64_t)blk * NF;
    auto* out = (__attribute__((address_space(1))) T*)ptr(ap->out) + (int64_t)blk * NC;
    // o_i = sum_k J[k][i] v_k, each handed to st(i, value)
    const auto line = [&](const T* v, auto st) {
#pragma unroll
      for (int i = 0; i < NPC; ++i) {
        T s = 0;
#pragma unroll
        for (int k = 0; k < NPF; ++k) s += J[k * NPC + i] * v[k];
        st(i, s);
      }
    };
    T v[NPF];
    if (tid < NPF * NPF) {
#pragma unroll
      for (int k = 0; k < NPF; ++k) v[k] = in[k * NPF * NPF + tid];
      line(v, [&](int i, T s) { A[i * NPF * NPF + tid] = s; });
    }
    __syncthreads();
    for (int q = tid; q < NPF * NPC; q += TH) {  // (i0, coarse i2)
      const int i2 = q / NPF, i0 = q - i2 * NPF;
#pragma unroll
      for (int k = 0; k < NPF; ++k) v[k] = A[(i2 * NPF + k) * NPF + i0];
      line(v, [&](int i, T s) { B[(i2 * NPC + i) * NPF + i0] = s; });
    }
    __syncthreads();
    for (int q = tid; q < NPC * NPC; q += TH) {
#pragma unroll
      for (int k = 0; k < NPF; ++k) v[k] = B[q * NPF + k];
      line(v, [&](int i, T s) { out[q * NPC + i] = s; });
    }
  } else {
    G* in = (G*)ptr(ap->in) + (int64_t)blk * NC;
    auto* out = (__attribute__((address_space(1))) T*)ptr(ap->out) + (int64_t)blk * NF;
    // o_i = sum_k J[i][k] v_k
    const auto line = [&](const T* v, auto st) {
#pragma unroll
      for (int i = 0; i < NPF; ++i) {
        T s = 0;
#pragma unroll
        for (int k = 0; k < NPC; ++k) s += J[i * NPC + k] * v[k];
        st(i, s);
      }
    };
    const bool has = tid < NPF * NPF;
    T u[NPF], v[NPC];
#pragma unroll
    for (int k = 0; k < NPF; ++k) u[k] = out[k * NPF * NPF + (has ? tid : 0)];
    for (int q = tid; q < NC; q += TH) A[q] = in[q];
    __syncthreads();
    for (int q = tid; q < NPC * NPC; q += TH) {
#pragma unroll
      for (int k = 0; k < NPC; ++k) v[k] = A[q * NPC + k];
      line(v, [&](int i, T s) { B[q * NPF + i] = s; });
    }
    __syncthreads();
    for (int q = tid; q < NPF * NPC; q += TH) {  // (i0, coarse i2)
      const int i2 = q / NPF, i0 = q - i2 * NPF;
#pragma unroll
      for (int k = 0; k < NPC; ++k) v[k] = B[(i2 * NPC + k) * NPF + i0];
      line(v, [&](int i, T s) { A[(i2 * NPF + i) * NPF + i0] = s; });
    }
    __syncthreads();
    if (has) {
#pragma unroll
      for (int k = 0; k < NPC; ++k) v[k] = A[k * NPF * NPF + tid];
      line(v, [&](int i, T s) { out[i * NPF * NPF + tid] = u[i] + s; });
    }
  }
}

// Blocks of one grid's transfer.
template <int DIM, int NPF>
int xfer_blocks(int n_elem) {
  constexpr int EPB = xfer_epb<NPF, DIM>();
  return (n_elem + EPB - 1) / EPB;
}

template <class T, int DIM, int NPF, int NPC, bool RESTRICT, bool BATCH>
void transfer_go(const XferArgs<T>& a, const BatchList<XferArgs<T>>& bl, int nblk, hipStream_t s) {
  if constexpr (DIM == 3 && xfer_lines<NPF>()) {
    hipLaunchKernelGGL((transfer3_kernel<T, NPF, NPC, RESTRICT, BATCH>), dim3(BATCH ? xcd_grid(nblk) : nblk),
                       dim3(round64(NPF * NPF)), 0, s, a, bl, nblk);
    return;
  }
  constexpr int EPB = xfer_epb<NPF, DIM>();
  const size_t shm = 2 * (size_t)EPB * ipow(NPF, DIM) * sizeof(T);
  if (shm > 65536)
    (void)hipFuncSetAttribute((const void*)transfer_kernel<T, DIM, NPF, NPC, RESTRICT, BATCH>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
  const int grid = BATCH ? xcd_grid(nblk) : nblk;
  hipLaunchKernelGGL((transfer_kernel<T, DIM, NPF, NPC, RESTRICT, BATCH>), dim3(grid), dim3(XFER_THREADS), shm, s,
                     a, bl, nblk);
}

template <class T, int DIM, int NPF, int NPC, bool RESTRICT>
int transfer_launch_t(const T* J, int n_elem, const T* in, T* out, const int* active, hipStream_t s) {
  XferArgs<T> a;
  a.J = J;
  a.n_elem = n_elem;
  a.in = in;
  a.out = out;
  a.active = active;
  transfer_go<T, DIM, NPF, NPC, RESTRICT, false>(a, BatchList<XferArgs<T>>{}, xfer_blocks<DIM, NPF>(n_elem), s);
  return 0;
}

// One launch over the transfers of many grids (same order pair and direction):
// ntot logical blocks, grid g's xfer_blocks in the range of bl.
template <class T, int DIM, int NPF, int NPC>
int transfer_batch_launch(bool restrict_, const BatchList<XferArgs<T>>& bl, int ntot, hipStream_t s) {
  if (restrict_) transfer_go<T, DIM, NPF, NPC, true, true>(XferArgs<T>{}, bl, ntot, s);
  else transfer_go<T, DIM, NPF, NPC, false, true>(XferArgs<T>{}, bl, ntot, s);
  return 0;
}

// ================================================================ dispatch (instantiated per T, DIM)
template <class T>
struct Fdm3Args;  // kernels_fdm3.hpp

template <class T>
struct ApplyArgs;  // kernels_apply.hpp
template <class T, int DIM>
struct Kern {
  // scratch: apply_big_scratch(n_elem, NP) elements (3D levels with NP = 33 only).
  // mode 3 (residual restricted to the coarser level, y coarse) returns -4 where
  // it is not built (large elements): the caller then runs mode 1 and transfer.
  static int apply(const LevelDev<T>& L, int mode, const T* x, const T* f, T* y, T* scratch, double* part,
                   int* nblk, hipStream_t s);
  // lat: the patches of this launch (all of them: PatchLat{}); large tiles
  // (3D P = 32) take only the whole partition
  static int fdm(const LevelDev<T>& L, int nd, int NA, int NL, const T* r, T* out, int npx, int npy,
                 int npz, const PatchBuf& pb, int waves, const PatchLat& lat, hipStream_t s);
  // wavefronts per block of a whole sweep's patch solve: 0 where the caller chooses
  // (fdm_kernel), else the one shape that its kernel is built for
  static int fdm_waves(int nd, int NA, int NL, int patches, const PatchBuf& pb);
  // patch-buffer layout of a level's sweep (np patches per direction, `step` node
  // positions apart along direction 1); whole = false: a launch over some of the
  // patches (strips of one patch)
  static PatchBuf patch_buf(int NP, int nd, int NA, int NL, const int* np, int step, bool whole);
  // u += the unweighted corrections of one patch-solve launch (disjoint patches)
  static int mult_update(const LevelDev<T>& L, int nd, int NA, int NL, const PatchLat& lat, int npx, int npy,
                         int npz, const PatchBuf& pb, const T* buf, T* u, hipStream_t s);
  // Batched launches (work lists over many grids, see BatchList): the same
  // kernels as above with per-grid arguments.  Block counts per grid:
  // apply_blocks, one per patch, combine_blocks, xfer_blocks.  -4 where the
  // template is not built.
  static int apply_blocks_of(int NP, int n_elem);
  static int combine_blocks_of(int NP, int n_elem);
  static int xfer_blocks_of(int NPF, int n_elem);
  static bool apply_in_lines(int NP, int n_elem);  // the form of a grid's apply
  static bool mode3_ok(const LevelDev<T>& L);
  static int apply_batch(int NP, int mode, bool lines, const BatchList<ApplyArgs<T>>& bl, int ntot, hipStream_t s);
  // pb: the longest strip of the launch's grids
  // (arguments: bl in 2D and where pb says that fdm_kernel solves the 3D tiles, else bl3)
  static int fdm_batch(int nd, int NA, int NL, const BatchList<FdmArgs<T>>& bl, const BatchList<Fdm3Args<T>>& bl3,
                       int ntot, const PatchBuf& pb, bool few, hipStream_t s);
  // maxc 0: the grids take combine3_kernel (arguments bl3), else combine_kernel (bl)
  static int combine_batch(int NP, int maxc, const BatchList<CombArgs<T>>& bl, const BatchList<Comb3Args<T>>& bl3,
                           int ntot, hipStream_t s);
  static int transfer_batch(int NPF, int NPC, bool restrict_, const BatchList<XferArgs<T>>& bl, int ntot,
                            hipStream_t s);
  static bool fdm_supported(int NA, int NL);
  // the order has compiled kernels (others run the run-time forms of kernels_gen.hpp)
  static bool order_compiled(int NP);
  // the tile's solve runs in LDS (not the large-tile stages through global memory)
  static bool fdm_in_lds(int NA, int NL);
  // assign: u = the overlap sum (u is zero on entry) instead of u += it
  static int combine(const LevelDev<T>& L, int nd, int NA, int NL, const T* buf, T* u, int npx,
                     int npy, int npz, const PatchBuf& pb, bool assign, hipStream_t s);
  // tmp: scratch of transfer_big_scratch(n_elem, NP, NPc) elements (3D levels with NP = 33 only)
  static int transfer(const LevelDev<T>& Lf, bool restrict_, const T* in, T* out, T* tmp, hipStream_t s);
  // Continuous spectral-element levels (lattice vectors, kernels_se.hpp).
  // ebuf: element-major scratch of n_elem * NP^DIM elements.  Modes 0 and 1.
  static int se_apply(const LevelDev<T>& L, int mode, const T* x, const T* f, T* y, T* ebuf, hipStream_t s);
  static int se_combine(const LevelDev<T>& L, int NA, const T* buf, T* u, const PatchBuf& pb, bool assign,
                        hipStream_t s);
  // ebuf (restriction only): n_elem * NPc^DIM elements
  static int se_transfer(const LevelDev<T>& Lf, const LevelDev<T>& Lc, bool restrict_, const T* in, T* out,
                         T* ebuf, hipStream_t s);
};

}  // namespace dgmg
