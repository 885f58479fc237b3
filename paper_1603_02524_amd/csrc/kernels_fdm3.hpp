// Patch solve by fast diagonalisation in 3D, tiles that fit in LDS (gfx950); sweeps of many
// patches of short lines take fdm_kernel (fdm_short_fits).
//
// One block solves a strip of K patches that follow each other along direction
// 1 (same indices in directions 0 and 2).  Their tiles overlap in node planes of
// direction 1, and patches of a strip share the eigenbases of directions 0 and
// 2, so each plane of the strip is transformed along directions 2 and 0 once,
// whatever number of patches hold it, and their weighted corrections are summed
// over the strip's patches before the way back: for the 16 x 13 x 13 tiles of
// P = 8 two patches have 22 planes instead of 26, and the patch buffer that the
// overlap sum reads shrinks likewise.
//
// Three phases with one barrier between them:
//   1  per plane (one wave): gather from the level vector straight into the
//      operand registers, transform along direction 2, through LDS within the
//      wave, transform along direction 0
//   2  per 16 lines of direction 1 (one wave, every patch of the strip in turn):
//      forward transform, division by the sum of the eigenvalues, backward
//      transform, weight of direction 1
//   3  per plane (one wave): back along direction 0, then direction 2, weights,
//      store
// A tile thus crosses LDS eight times instead of twelve, with three barriers instead of
// seven (one pass per direction and way with a gather and a scatter stage, the form
// before).
//
// What bounds it: instruction issue.  The matrix products and the FP64 vector
// instructions (eigenvalue division, rank-one tails) share the SIMDs' time and hardly
// overlap; of a block's 39 k cycles (16 x 13 x 13 tiles, FP64, strips of two, three blocks
// per compute unit) 6 k are the start (arguments, tables and first residual values), 12 k
// phase 1, 15 k phase 2, 7 k phase 3.  Measured per launch, before -> now (event pairs,
// which add some 8 us): 16 x 13 x 13 on 4352 patches FP64 83 -> 73 us, on 33792 patches
// FP32 332 -> 226 us; 8 x 9 x 9 on 4352 patches FP64 29 -> 27 us; 11^3 on 4096 patches FP64
// 44 -> 36 us.  Not faster: 16x16x4 products (the launch within 2 %), two or four waves per
// SIMD instead of three, matrices read from global memory by each wave (its vector memory
// path was then two thirds busy).
#pragma once

#include <initializer_list>
#include <type_traits>

#include "kernels.hpp"

namespace dgmg {

// ---------------------------------------------------------------- line transforms
// The 1D matrix of a transform out_j = sum_k M[k][j] v_k (M row-major LEN x LEN)
// as matrix-core operand.  The data are the B operand: lane (li, lk) = (lane %
// 16, lane / 16) supplies values k = 4 ks + lk of line li and receives rows j =
// 4 r + lk of the same line, so that one transform's results are the next one's
// operands.
//
// FP64: 4x4x4 products, four blocks of four lines with the same matrix block.
// With every compute unit busy they sustain 75 TFLOP/s, the 16x16x4 product only
// 49 (it stalls chip-wide, not on one unit), and lines need padding to a
// multiple of 4 only.  Lines of 4 m + 1 values take their last value as a
// rank-one update on the VALU instead of a fourth product of four that is 3/4
// padding.
template <class T, int LEN>
struct FdmOp;

template <int LEN>
struct FdmOp<double, LEN> {
  static constexpr int KC = (LEN + 3) / 4, AC = KC;
  static constexpr bool TAIL = LEN % 4 == 1 && LEN > 4;
  static constexpr int KM = TAIL ? KC - 1 : KC;
  double a[KC][KM];
  double t[TAIL ? KC : 1];
  template <int SK, int SJ>
  __device__ __forceinline__ void load(const double* M) {
    const int lane = threadIdx.x & 63, i = lane & 3, lk = lane >> 4;
#pragma unroll
    for (int jc = 0; jc < KC; ++jc)
#pragma unroll
      for (int ks = 0; ks < KM; ++ks) {
        const int j = 4 * jc + i, k = 4 * ks + lk;
        a[jc][ks] = M[k * SK + j * SJ];
      }
    if constexpr (TAIL) {
#pragma unroll
      for (int jc = 0; jc < KC; ++jc) {
        const int j = 4 * jc + lk;
        t[jc] = M[(LEN - 1) * SK + j * SJ];
      }
    }
  }
  __device__ __forceinline__ void apply(const double* v, double vl, double* acc) const {
#pragma unroll
    for (int jc = 0; jc < KC; ++jc) acc[jc] = 0.0;
#pragma unroll
    for (int ks = 0; ks < KM; ++ks)
#pragma unroll
      for (int jc = 0; jc < KC; ++jc) acc[jc] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[jc][ks], v[ks], acc[jc], 0, 0, 0);
    if constexpr (TAIL) {
#pragma unroll
      for (int jc = 0; jc < KC; ++jc) acc[jc] = __builtin_fma(t[jc], vl, acc[jc]);
    }
  }
};

// FP32: 16x16x4 products; row i of the product is output j = 4 (i % 4) + i / 4, so
// that result register r of lane (li, lk) is j = 4 r + lk here too.
template <int LEN>
struct FdmOp<float, LEN> {
  static constexpr int KC = (LEN + 3) / 4, NB = (LEN + 15) / 16, AC = 4 * NB;
  static constexpr bool TAIL = false;
  static constexpr int KM = KC;
  float a[NB][KC];
  template <int SK, int SJ>
  __device__ __forceinline__ void load(const float* M) {
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int ks = 0; ks < KC; ++ks) {
        const int j = 16 * nb + 4 * (li & 3) + (li >> 2), k = 4 * ks + lk;
        if constexpr (fdm3_padded<float>(LEN)) {
          a[nb][ks] = M[k * SK + j * SJ];
        } else {  // a valid index, zero outside the matrix
          const float v = M[imin(k, LEN - 1) * SK + imin(j, LEN - 1) * SJ];
          a[nb][ks] = k < LEN && j < LEN ? v : 0.0f;
        }
      }
  }
  __device__ __forceinline__ void apply(const float* v, float, float* acc) const {
    typedef float acc_t __attribute__((ext_vector_type(4)));
    acc_t c[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) c[nb] = acc_t{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < KC; ++ks)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) c[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[nb][ks], v[ks], c[nb], 0, 0, 0);
#pragma unroll
    for (int r = 0; r < AC; ++r) acc[r] = c[r / 4][r % 4];
  }
};

// Values k = 4 ks + lk of a line in LDS (past its end: some value of the line, the
// matrix is zero there), and its last value where the transform takes it apart.
template <class T, int LEN, int STRIDE>
__device__ __forceinline__ void fdm_line_read(const T* p, int lk, T* v, T& vl) {
  using Op = FdmOp<T, LEN>;
#pragma unroll
  for (int ks = 0; ks < Op::KM; ++ks) v[ks] = p[(4 * ks + 3 < LEN ? 4 * ks + lk : imin(4 * ks + lk, LEN - 1)) * STRIDE];
  if constexpr (Op::TAIL) vl = p[(LEN - 1) * STRIDE];
}
template <class T, int LEN, int STRIDE>
__device__ __forceinline__ void fdm_line_write(T* p, int lk, const T* acc) {
#pragma unroll
  for (int r = 0; r < FdmOp<T, LEN>::KC; ++r)
    if (4 * r + 3 < LEN || 4 * r + lk < LEN) p[(4 * r + lk) * STRIDE] = acc[r];
}

// LDS written by some lanes of a wave is read by others of the same wave: the
// wave's LDS accesses are executed in order, so the compiler only has to keep them.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------- tile geometry
template <int NA, int NL, int ND>
struct Fdm3Shape {
  static constexpr int LX = ND == 0 ? NA : NL, LY = ND == 1 ? NA : NL, LZ = ND == 2 ? NA : NL;
  static constexpr int PX = LX | 1;    // odd row pitch: lines across rows spread over the banks
  static constexpr int PS = LZ * PX;   // plane pitch
};
// n items in batches of at most B (a compile-time count each).
template <int B, class F>
__device__ __forceinline__ void fdm3_batches(int n, F f) {
  int t = 0;
  for (; t + B <= n; t += B) f(std::integral_constant<int, B>(), t);
  if constexpr (B > 3)
    if (n - t == 3) f(std::integral_constant<int, 3>(), t);
  if constexpr (B > 2)
    if (n - t == 2) f(std::integral_constant<int, 2>(), t);
  if constexpr (B > 1)
    if (n - t == 1) f(std::integral_constant<int, 1>(), t);
}
constexpr int fdm3_planes(int NA, int NL) { return imax(NA, NL) <= 9 ? 4 : (imax(NA, NL) <= 16 ? 3 : 1); }
// Dynamic LDS of a strip of K patches, `step` planes apart.
template <class T, int NA, int NL, int ND>
constexpr size_t fdm3_shmem(int K, int step) {
  using S = Fdm3Shape<NA, NL, ND>;
  return (((size_t)(K - 1) * step + S::LY) * S::PS + fdm3_image<T>(S::LX) + fdm3_image<T>(S::LZ) +
          (size_t)K * fdm3_image<T>(S::LY) + 2 * (S::LX + S::LZ + (size_t)K * S::LY)) *
         sizeof(T);
}
// Strips of several patches are built for tiles of at most 16 values per line.
constexpr bool fdm3_strips(int NA, int NL) { return imax(NA, NL) <= 16; }
// Waves per block: 4, and 8 for tiles of which a compute unit holds at most two.
template <class T, int NA, int NL>
constexpr int fdm3_waves() {
  return (size_t)NA * NL * NL * sizeof(T) > 50 * 1024 ? 8 : 4;
}
// Waves per SIMD asked of the compiler (register budget): four blocks of 4 waves
// per compute unit for the small tiles, what the LDS allows for the others.
template <class T, int NA, int NL>
constexpr int fdm3_occupancy() {
  return imax(NA, NL) <= 9 ? 4 : (imax(NA, NL) <= 16 ? (sizeof(T) == 4 ? 4 : 3) : 2);
}

// Arguments of a launch, only what the kernel reads, the tables chosen by the host
// for the sweep's normal: a block's start is a chain of scalar loads and scalar
// arithmetic that every wave waits for, so both are kept short.
template <class T>
struct Fdm3Args {
  const T* r = nullptr;         // residual (level vector)
  T* out = nullptr;             // weighted corrections, one tile per strip
  const T* img[3] = {nullptr, nullptr, nullptr};  // per direction and patch: eigenvectors (padded), eigenvalues,
  const T* lam[3] = {nullptr, nullptr, nullptr};  // weights; offsets into the level vector of the positions
  const T* w[3] = {nullptr, nullptr, nullptr};    // (-1: outside), patch p starting at position p step
  const int* gp[3] = {nullptr, nullptr, nullptr};
  const int* active = nullptr;
  int npx = 1, npy = 1, nsy = 1, nblk = 1;
  int K = 1, step = 0;
  uint32_t mx = 0, my = 0;  // divisions by npx and nsy
  PatchLat lat;
};
template <class T>
Fdm3Args<T> fdm3_args(const LevelDev<T>& L, int nd, const T* r, T* out, int npx, int npy, int npz,
                      const PatchBuf& pb, const PatchLat& lat) {
  Fdm3Args<T> a;
  a.r = r;
  a.out = out;
  for (int d = 0; d < 3; ++d) {
    const DirDev<T>& dd = L.dir[d];
    a.img[d] = d == nd ? dd.img_fc : dd.img_ec;
    a.lam[d] = d == nd ? dd.lam_fc : dd.lam_ec;
    a.w[d] = d == nd ? dd.w_fc : dd.w_ec;
    a.gp[d] = d == nd ? dd.gp_fc : dd.gp_ec;
  }
  a.active = L.active;
  a.npx = npx;
  a.npy = npy;
  a.nsy = (npy + pb.K - 1) / pb.K;
  a.nblk = npx * a.nsy * npz;
  a.K = pb.K;
  a.step = pb.step;
  a.mx = div_magic(a.nblk, npx);
  a.my = div_magic(a.nblk, a.nsy);
  a.lat = lat;
  return a;
}

// The tile's solve runs here: a patch, with its matrices and a work list's arguments, in LDS
// whatever the normal (FP32 33 x 33 x 33, the largest: 158412 + 176 bytes of 163840).
template <class T, int NA, int NL>
constexpr bool fdm3_fits() {
  size_t most = 0;
  for (const size_t b : {fdm3_shmem<T, NA, NL, 0>(1, 0), fdm3_shmem<T, NA, NL, 1>(1, 0), fdm3_shmem<T, NA, NL, 2>(1, 0)})
    most = b > most ? b : most;
  return most + (sizeof(Fdm3Args<T>) + 15) / 16 * 16 <= LDS_BYTES;
}

// BATCH: the arguments come from the work list bl (ntot logical blocks in all)
template <class T, int NA, int NL, int ND, bool BATCH = false>
__global__ void __launch_bounds__((64 * fdm3_waves<T, NA, NL>()))
    __attribute__((amdgpu_waves_per_eu((fdm3_occupancy<T, NA, NL>()))))
    fdm3_kernel(Fdm3Args<T> a0, BatchList<Fdm3Args<T>> bl, int ntot) {
  using S = Fdm3Shape<NA, NL, ND>;
  constexpr int LX = S::LX, LY = S::LY, LZ = S::LZ, PX = S::PX, PS = S::PS;
  constexpr int NW = fdm3_waves<T, NA, NL>();
  constexpr int NBX = (LX + 15) / 16, NBZ = (LZ + 15) / 16;  // 16-line blocks of a plane, by line direction
  constexpr int LINES = LX * LZ, MBY = (LINES + 15) / 16, NBW = (MBY + NW - 1) / NW;
  using OpX = FdmOp<T, LX>;
  using OpY = FdmOp<T, LY>;
  using OpZ = FdmOp<T, LZ>;
  constexpr bool STRIP = fdm3_strips(NA, NL);  // strips of more than one patch are built
  constexpr int OVR = (LY / 2 + 3) / 4;        // registers for the planes shared by two patches (at most LY / 2)
  // planes and line blocks that a wave takes at once (independent product chains), as registers allow
  constexpr int PB = fdm3_planes(NA, NL), LB = sizeof(T) == 4 ? 2 : 1;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ __align__(16) int sargs_raw[BATCH ? sizeof(Fdm3Args<T>) / sizeof(int) : 1];
  const Fdm3Args<T>* ap;
  int pid = 0;
  if constexpr (BATCH) {
    const int b = xcd_block(ntot);
    if (b < 0) return;
    Fdm3Args<T>* sargs = reinterpret_cast<Fdm3Args<T>*>(sargs_raw);
    pid = batch_pick(bl, b, sargs);
    ap = sargs;
  } else {
    ap = &a0;
  }
  // every argument into scalar registers by one group of loads (left to itself the
  // compiler loads each before its use: a dozen round trips in a row)
  const auto uni = [](int v) { return BATCH ? __builtin_amdgcn_readfirstlane(v) : v; };
  const auto ptr = [](auto* q) { return BATCH ? sgpr_ptr(q) : q; };
  const T *i0 = ptr(ap->img[0]), *i1 = ptr(ap->img[1]), *i2 = ptr(ap->img[2]);
  const T *l0 = ptr(ap->lam[0]), *l1 = ptr(ap->lam[1]), *l2 = ptr(ap->lam[2]);
  const T *w0 = ptr(ap->w[0]), *w1 = ptr(ap->w[1]), *w2 = ptr(ap->w[2]);
  const int *g0 = ptr(ap->gp[0]), *g1 = ptr(ap->gp[1]), *g2 = ptr(ap->gp[2]);
  const T* rr0 = ptr(ap->r);
  T* oo0 = ptr(ap->out);
  const int* act = ptr(ap->active);
  int K = uni(ap->K), step = uni(ap->step), npx = uni(ap->npx), npy = uni(ap->npy), nsy = uni(ap->nsy);
  int nblk = uni(ap->nblk);
  uint32_t mx = uni(ap->mx), my = uni(ap->my);
  int st0 = uni(ap->lat.start[0]), st1 = uni(ap->lat.start[1]), st2 = uni(ap->lat.start[2]);
  int sr0 = uni(ap->lat.stride[0]), sr1 = uni(ap->lat.stride[1]), sr2 = uni(ap->lat.stride[2]);
  if constexpr (!BATCH) {
    asm volatile("" : "+s"(i0), "+s"(i1), "+s"(i2), "+s"(l0), "+s"(l1), "+s"(l2), "+s"(w0), "+s"(w1), "+s"(w2),
                 "+s"(g0), "+s"(g1), "+s"(g2), "+s"(rr0), "+s"(oo0), "+s"(act));
    asm volatile("" : "+s"(K), "+s"(step), "+s"(npx), "+s"(npy), "+s"(nsy), "+s"(mx), "+s"(my), "+s"(st0), "+s"(st1),
                 "+s"(st2), "+s"(sr0), "+s"(sr1), "+s"(sr2), "+s"(nblk));
    pid = xcd_block(nblk);
    if (pid < 0) return;
  }
  using G = const __attribute__((address_space(1))) T;  // global memory
  using GI = const __attribute__((address_space(1))) int;
  G *img0 = (G*)i0, *img1 = (G*)i1, *img2 = (G*)i2, *lam0 = (G*)l0, *lam1 = (G*)l1, *lam2 = (G*)l2;
  G *wgt0 = (G*)w0, *wgt1 = (G*)w1, *wgt2 = (G*)w2, *r = (G*)rr0;
  GI *gp0 = (GI*)g0, *gp1 = (GI*)g1, *gp2 = (GI*)g2;
  auto* out0 = (__attribute__((address_space(1))) T*)oo0;
  if (act != nullptr && *(GI*)act == 0) return;
  pid = uni(pid);
  const int pq = uni(div_by(pid, npx, mx)), sx = pid - pq * npx;
  const int sz = uni(div_by(pq, nsy, my)), sy = pq - sz * nsy;
  const int p0 = st0 + sr0 * sx, p2 = st2 + sr2 * sz;
  const int p1 = st1 + sr1 * sy * K;  // first patch of the strip (those of longer strips follow each other)
  const int kact = imin(K, npy - sy * K);
  const int np = (kact - 1) * step + LY;  // planes of the strip
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lk = lane >> 4;
  // the wave that gets one more plane or line block than the others differs from block to block
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wv = (wave + pid) & (NW - 1);
  static_assert((NW & (NW - 1)) == 0, "power of two");
  // lane t holds the offset of the wave's t-th plane sp = wv + NW t
  const int plane_off = gp1[p1 * step + imin(wv + NW * lane, np - 1)];
  const int nt = (np - wv + NW - 1) / NW;  // planes of this wave
  constexpr int NV = OpZ::KM + (OpZ::TAIL ? 1 : 0);
  GI *gox = gp0 + p0 * step, *goz = gp2 + p2 * step;
  int off[NBX][NV], gz[NV];  // -1: outside a Dirichlet domain
#pragma unroll
  for (int xb = 0; xb < NBX; ++xb) off[xb][0] = gox[imin(16 * xb + li, LX - 1)];
#pragma unroll
  for (int ks = 0; ks < NV; ++ks) gz[ks] = goz[ks < OpZ::KM ? imin(4 * ks + lk, LZ - 1) : LZ - 1];
  bool full = true;  // no position outside the domain (then nothing to mask but whole planes)
  const auto offsets = [&]() {
#pragma unroll
    for (int xb = 0; xb < NBX; ++xb) {
      const int gx = off[xb][0];
#pragma unroll
      for (int ks = 0; ks < NV; ++ks) {
        const bool in = (gx | gz[ks]) >= 0;
        off[xb][ks] = in ? gx + gz[ks] : -1;
        full = full && in;
      }
    }
    full = __all(full);
  };
  T v[PB][NBX][NV];
  int gy[PB];
  const auto gather = [&](int t0) {  // past the wave's planes: its last one again
#pragma unroll
    for (int c = 0; c < PB; ++c) {
      gy[c] = __builtin_amdgcn_readlane(plane_off, imin(t0 + c, imax(nt - 1, 0)));
      G* rp = r + imax(gy[c], 0);
#pragma unroll
      for (int xb = 0; xb < NBX; ++xb)
#pragma unroll
        for (int ks = 0; ks < NV; ++ks) v[c][xb][ks] = rp[imax(off[xb][ks], 0)];
    }
  };
  // LDS: the matrices of directions 0 and 2 and of the patches along direction 1 (used as
  // S and as S^T), eigenvalues and weights in the same order, the tile
  constexpr int QX = fdm3_pitch<T>(LX), QY = fdm3_pitch<T>(LY), QZ = fdm3_pitch<T>(LZ);
  constexpr int IX = fdm3_image<T>(LX), IY = fdm3_image<T>(LY), IZ = fdm3_image<T>(LZ), SY = IY;
  T* smx = reinterpret_cast<T*>(smem_raw);
  T* smz = smx + IX;
  T* smy = smz + IZ;
  T* slx = smy + K * IY;
  T* slz = slx + LX;
  T* sly = slz + LZ;
  T* swx = sly + K * LY;
  T* swz = swx + LX;
  T* swy = swz + LZ;
  T* tile = swy + K * LY;
  {
    typedef int vec __attribute__((ext_vector_type(4)));
    constexpr int PV = 16 / sizeof(T), VX = IX / PV, VZ = IZ / PV, VY = IY / PV;  // 16-byte pieces
    static_assert(IX % PV == 0 && IY % PV == 0 && IZ % PV == 0, "whole pieces");
    // each wave copies a part of its own (matrix x, z, half of y), so that the choice is scalar
    const int role = wave & 3;
    int n = role == 0 ? VX : (role == 1 ? VZ : kact * VY), at = 0;
    G* from = role == 0 ? img0 + (int64_t)p0 * IX : (role == 1 ? img2 + (int64_t)p2 * IZ : img1 + (int64_t)p1 * IY);
    if (role >= 2) {
      const int h = (n + 1) >> 1;
      at = role == 3 ? h : 0;
      n = role == 3 ? n - h : h;
    }
    if (NW == 8) {
      const int h = (n + 1) >> 1;
      at += wave >= 4 ? h : 0;
      n = wave >= 4 ? n - h : h;
    }
    using GV = const __attribute__((address_space(1))) vec;
    GV* src = (GV*)from + at;
    vec* dst = reinterpret_cast<vec*>(smem_raw) + ((role == 0 ? 0 : (role == 1 ? VX : VX + VZ)) + at);
    constexpr int CV = 3;
    vec m[CV];
#pragma unroll
    for (int c = 0; c < CV; ++c) m[c] = src[imin(lane + 64 * c, imax(n - 1, 0))];
    // eigenvalues and weights: waves 0, 1, 2 for directions 0, 2, 1
    G* lam = wave == 0 ? lam0 + p0 * LX : (wave == 1 ? lam2 + p2 * LZ : lam1 + p1 * LY);
    G* wgt = wave == 0 ? wgt0 + p0 * LX : (wave == 1 ? wgt2 + p2 * LZ : wgt1 + p1 * LY);
    const int nl = wave == 0 ? LX : (wave == 1 ? LZ : (wave == 2 ? kact * LY : 0));
    const int to = wave == 0 ? 0 : (wave == 1 ? LX : LX + LZ);
    T l = T(0), w = T(0);
    if (lane < nl) {
      l = lam[lane];
      w = wgt[lane];
    }
    offsets();
    gather(0);
#pragma unroll
    for (int c = 0; c < CV; ++c)
      if (lane + 64 * c < n) dst[lane + 64 * c] = m[c];
    for (int q = lane + 64 * CV; q < n; q += 64) dst[q] = src[q];
    if (lane < nl) {
      slx[to + lane] = l;
      swx[to + lane] = w;
    }
    for (int q = lane + 64; q < nl; q += 64) {
      slx[to + q] = lam[q];
      swx[to + q] = wgt[q];
    }
  }

  // ---- phase 1: planes forward along directions 2 and 0
  {
    __syncthreads();  // the matrices
    OpZ Mz;
    Mz.template load<QZ, 1>(smz);
    OpX Mx;
    Mx.template load<QX, 1>(smx);
    const auto planes = [&](auto N, int t0) {
      constexpr int C = decltype(N)::value;
      T az[C][NBX][OpZ::AC];
      if (!full) {
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
          for (int xb = 0; xb < NBX; ++xb)
#pragma unroll
            for (int ks = 0; ks < NV; ++ks) v[c][xb][ks] = off[xb][ks] >= 0 ? v[c][xb][ks] : T(0);
      }
#pragma unroll
      for (int c = 0; c < C; ++c) {
        if (gy[c] < 0) {
#pragma unroll
          for (int xb = 0; xb < NBX; ++xb)
#pragma unroll
            for (int ks = 0; ks < NV; ++ks) v[c][xb][ks] = T(0);
        }
      }
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int xb = 0; xb < NBX; ++xb) Mz.apply(v[c][xb], v[c][xb][NV - 1], az[c][xb]);
      if (t0 + C < nt) gather(t0 + C);
      T* pl = tile + (wv + NW * t0) * PS;
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int xb = 0; xb < NBX; ++xb)
          if ((16 * xb + 15 < LX) || 16 * xb + li < LX)
            fdm_line_write<T, LZ, PX>(pl + c * NW * PS + 16 * xb + li, lk, az[c][xb]);
      wave_lds_order();
      T u[C][NBZ][OpX::KM], ul[C][NBZ], ax[C][NBZ][OpX::AC];
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int zb = 0; zb < NBZ; ++zb)
          fdm_line_read<T, LX, 1>(pl + c * NW * PS + imin(16 * zb + li, LZ - 1) * PX, lk, u[c][zb], ul[c][zb]);
      wave_lds_order();
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int zb = 0; zb < NBZ; ++zb) Mx.apply(u[c][zb], ul[c][zb], ax[c][zb]);
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int zb = 0; zb < NBZ; ++zb)
          if ((16 * zb + 15 < LZ) || 16 * zb + li < LZ)
            fdm_line_write<T, LX, 1>(pl + c * NW * PS + (16 * zb + li) * PX, lk, ax[c][zb]);
    };
    fdm3_batches<PB>(nt, planes);
  }
  __syncthreads();

  // ---- phase 2: lines of direction 1, patch after patch
  {
    const int wl = (wv + NW / 2) % NW;
    T keep[STRIP ? NBW : 1][OVR];  // the next patch's first planes, before this patch's results overwrite them
    const int ov = LY - step;      // planes shared with the next (previous) patch
    for (int i = 0; i < kact; ++i) {
      const T* Sy = smy + i * SY;
      T ly[OpY::KC], wy[OpY::KC];
#pragma unroll
      for (int rr = 0; rr < OpY::KC; ++rr) {
        const int y = 4 * rr + 3 < LY ? 4 * rr + lk : imin(4 * rr + lk, LY - 1);
        ly[rr] = sly[i * LY + y];
        wy[rr] = swy[i * LY + y];
      }
      T* tp = tile + i * step * PS;
      OpY M;
      // the wave's line blocks t0 .. t0 + N - 1 (16 lines each; lines past the last one are
      // computed and dropped); way 0: forward and scaled, 1: backward and weighted, 2: both
      const auto lines = [&](auto N, int t0, int way) {
        constexpr int C = decltype(N)::value;
        T v[C][imax(OpY::KM, OVR)], vl[C], acc[C][OpY::AC];
        T* ln[C];
        bool in[C];
        T lx[C], lz[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
          const int q = 16 * (wl + NW * (t0 + c)) + li, qc = imin(q, LINES - 1), z = qc / LX, x = qc - z * LX;
          ln[c] = tp + z * PX + x;
          lx[c] = slx[x];
          lz[c] = slz[z];
          in[c] = q < LINES;
          fdm_line_read<T, LY, PS>(ln[c], lk, v[c], vl[c]);
          if constexpr (STRIP) {
            if (i > 0) {
#pragma unroll
              for (int k = 0; k < OVR; ++k)
                if (4 * k + lk < ov) v[c][k] = keep[c][k];
            }
            if (i + 1 < kact) {
#pragma unroll
              for (int k = 0; k < OVR; ++k) keep[c][k] = ln[c][(step + imin(4 * k + lk, LY - step - 1)) * PS];
            }
          }
        }
        wave_lds_order();
        if (way != 1) {
#pragma unroll
          for (int c = 0; c < C; ++c) M.apply(v[c], vl[c], acc[c]);
#pragma unroll
          for (int c = 0; c < C; ++c)
#pragma unroll
            for (int rr = 0; rr < OpY::KC; ++rr) acc[c][rr] = div_nr(acc[c][rr], (lx[c] + ly[rr]) + lz[c]);
        }
        if (way == 2) {
          M.template load<1, QY>(Sy);
#pragma unroll
          for (int c = 0; c < C; ++c) {
#pragma unroll
            for (int k = 0; k < OpY::KM; ++k) v[c][k] = acc[c][k];
            if constexpr (OpY::TAIL) vl[c] = __shfl(acc[c][OpY::KC - 1], li, 64);  // value LY - 1: lane (li, 0)
          }
        }
        if (way != 0) {
#pragma unroll
          for (int c = 0; c < C; ++c) M.apply(v[c], vl[c], acc[c]);
        }
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
          for (int rr = 0; rr < OpY::KC; ++rr) {
            const int y = 4 * rr + lk;
            if ((4 * rr + 3 < LY || y < LY) && in[c]) {
              T res = way == 0 ? acc[c][rr] : wy[rr] * acc[c][rr];
              if constexpr (STRIP)
                if (i > 0 && y < ov) res += ln[c][y * PS];
              ln[c][y * PS] = res;
            }
          }
        wave_lds_order();
      };
      const int nb = (MBY - wl + NW - 1) / NW;
      if constexpr (STRIP) {
        M.template load<QY, 1>(Sy);
        if (nb == NBW) lines(std::integral_constant<int, NBW>(), 0, 2);
        else if constexpr (NBW > 1) lines(std::integral_constant<int, NBW - 1>(), 0, 2);
      } else {  // one matrix at a time over all lines (strips of one patch)
        M.template load<QY, 1>(Sy);
        fdm3_batches<LB>(nb, [&](auto N, int t0) { lines(N, t0, 0); });
        M.template load<1, QY>(Sy);
        fdm3_batches<LB>(nb, [&](auto N, int t0) { lines(N, t0, 1); });
      }
    }
  }
  __syncthreads();

  // ---- phase 3: planes back along directions 0 and 2, weights, store
  {
    OpX Mx;
    Mx.template load<1, QX>(smx);
    OpZ Mz;
    Mz.template load<1, QZ>(smz);
    T w[NBX][OpZ::KC];
#pragma unroll
    for (int xb = 0; xb < NBX; ++xb)
#pragma unroll
      for (int rr = 0; rr < OpZ::KC; ++rr)
        w[xb][rr] = swx[imin(16 * xb + li, LX - 1)] * swz[imin(4 * rr + lk, LZ - 1)];
    auto* dst = out0 + (int64_t)pid * ((K - 1) * step + LY) * LINES;
    const auto planes = [&](auto N, int t0) {
      constexpr int C = decltype(N)::value;
      T* pl = tile + (wv + NW * t0) * PS;
      T u[C][NBZ][OpX::KM], ul[C][NBZ], ax[C][NBZ][OpX::AC];
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int zb = 0; zb < NBZ; ++zb)
          fdm_line_read<T, LX, 1>(pl + c * NW * PS + imin(16 * zb + li, LZ - 1) * PX, lk, u[c][zb], ul[c][zb]);
      wave_lds_order();
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int zb = 0; zb < NBZ; ++zb) Mx.apply(u[c][zb], ul[c][zb], ax[c][zb]);
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int zb = 0; zb < NBZ; ++zb)
          if ((16 * zb + 15 < LZ) || 16 * zb + li < LZ)
            fdm_line_write<T, LX, 1>(pl + c * NW * PS + (16 * zb + li) * PX, lk, ax[c][zb]);
      wave_lds_order();
      T s[C][NBX][OpZ::KM], sl[C][NBX], az[C][NBX][OpZ::AC];
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int xb = 0; xb < NBX; ++xb)
          fdm_line_read<T, LZ, PX>(pl + c * NW * PS + imin(16 * xb + li, LX - 1), lk, s[c][xb], sl[c][xb]);
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int xb = 0; xb < NBX; ++xb) Mz.apply(s[c][xb], sl[c][xb], az[c][xb]);
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int xb = 0; xb < NBX; ++xb)
          if ((16 * xb + 15 < LX) || 16 * xb + li < LX) {
            auto* o = dst + (int64_t)(wv + NW * (t0 + c)) * LINES + 16 * xb + li;
#pragma unroll
            for (int rr = 0; rr < OpZ::KC; ++rr)
              if (4 * rr + 3 < LZ || 4 * rr + lk < LZ) o[(4 * rr + lk) * LX] = w[xb][rr] * az[c][xb][rr];
          }
    };
    fdm3_batches<PB>(nt, planes);
  }
}

template <class T, int NA, int NL, int ND, bool BATCH>
int fdm3_launch_nd(const Fdm3Args<T>& a, const BatchList<Fdm3Args<T>>& bl, int nlog, hipStream_t s) {
  static_assert(fdm3_fits<T, NA, NL>(), "a patch and its matrices fit the LDS");
  const size_t shm = fdm3_shmem<T, NA, NL, ND>(a.K, a.step);
  if (shm > 65536 && hipFuncSetAttribute((const void*)fdm3_kernel<T, NA, NL, ND, BATCH>,
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm) != hipSuccess)
    return -4;
  hipLaunchKernelGGL((fdm3_kernel<T, NA, NL, ND, BATCH>), dim3(xcd_grid(nlog)), dim3(64 * fdm3_waves<T, NA, NL>()), shm,
                     s, a, bl, nlog);
  return 0;
}

// Batched: a's K and step are those of the longest strip of the launch (its LDS), bl
// holds each grid's own arguments.
template <class T, int NA, int NL, bool BATCH>
int fdm3_go(int nd, const Fdm3Args<T>& a, const BatchList<Fdm3Args<T>>& bl, int nlog, hipStream_t s) {
  if (nd < 0) {
    if constexpr (NA == NL) return fdm3_launch_nd<T, NA, NL, -1, BATCH>(a, bl, nlog, s);
    else return -4;
  }
  if (nd == 0) return fdm3_launch_nd<T, NA, NL, 0, BATCH>(a, bl, nlog, s);
  if (nd == 1) return fdm3_launch_nd<T, NA, NL, 1, BATCH>(a, bl, nlog, s);
  return fdm3_launch_nd<T, NA, NL, 2, BATCH>(a, bl, nlog, s);
}

// Patches per strip of a whole-partition sweep (np patches per direction, `step`
// planes apart, tile NA, NL, normal nd): a power of two.  Longer strips share more
// planes (and shrink the patch buffer) but need more LDS and leave fewer, longer blocks:
// three blocks per compute unit have to fit (52 KB each), and the strips have to be at
// least 512 K (128 K for lines of up to 4 values, whose planes are little work: 3 x 3 x 3 FP64
// on 6156 patches 10.0 -> 8.7 us with K = 4 instead of 2).  Measured (us per launch for K = 1 / 2 / 4): 16 x 13 x 13 FP64 on 4352
// patches 85 / 73 / 83 (one block per unit at 4), FP32 on 33792 patches 284 / 233 / 226;
// 8 x 9 x 9 FP64 on 4352 patches 32 / 27 / 28; 11^3 FP64 on 4096 patches 41 / 36 / 35.
template <class T>
int fdm3_strip(int NA, int NL, int nd, const int* np, int step) {
  const int LX = nd == 0 ? NA : NL, LY = nd == 1 ? NA : NL, LZ = nd == 2 ? NA : NL;
  if (!fdm3_strips(NA, NL) || LY > 2 * step) return 1;
  int best = 1;
  for (int K : {2, 4, 8}) {
    if (K > np[1] || (int64_t)np[0] * ((np[1] + K - 1) / K) * np[2] < (NL <= 4 ? 128 : 512) * (int64_t)K) break;
    const size_t lds = ((size_t)((K - 1) * step + LY) * LZ * (LX | 1) + fdm3_image<T>(LX) + fdm3_image<T>(LZ) +
                        (size_t)K * fdm3_image<T>(LY) + 2 * (LX + LZ + (size_t)K * LY)) * sizeof(T);
    if (lds > 52 * 1024) break;
    best = K;
  }
  return best;
}

}  // namespace dgmg
