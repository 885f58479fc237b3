// Operator apply on DG levels (compiled orders).
// y = A x (MODE 0), y = f - A x (MODE 1), y = A x plus per-block partial x.y (MODE 2),
// or the restriction of f - A x to the next coarser level, y = (J^T x J^T x J^T)(f - A x)
// per element (MODE 3: the V-cycle's residual and restriction in one pass; the
// fine residual stays in LDS and the transfer's contraction passes run on it).
//
// 3D: a block takes apply_epb consecutive elements and goes through the directions one
// after the other; in each, a thread owns one line of one element: its values from LDS,
// the two neighbours' lines (traces and normal derivatives, eq. (L:generic)), the rows of
// the 1D matrix from scalar registers.  Each node receives one contribution per
// direction, added up in LDS in direction order; the last direction's lanes run along
// the vector, so they read f and write y themselves.
// Bound: memory in FP32, the vector instructions and their waits in FP64.  The line
// form below (lines of all directions at once, the direction chosen per lane, every
// neighbour line from global memory at the line's stride) issued more than twice the
// instructions, and its lines along direction 0 touched one cache line per lane and load;
// here the direction and so every stride is a constant, direction 0 sees its neighbours
// through LDS (coalesced loads), and a block loads its arguments in one group.  Residual,
// line form and this: 32^3 P = 8 FP32 132 -> 86 us (3.3 TB/s), 16^3 P = 8 FP64 27.6 -> 22.3 us
// (3.2 TB/s), 9x7x11 P = 12 FP32 16.3 -> 11.8 and FP64 30 -> 18.3 us, 7x9x6 P = 16 FP64
// 53.5 -> 42 us.
// 2D: a thread per node (apply2_kernel).  Large 2D and small 3D grids take the line form
// (apply_lines).
#pragma once

#include "kernels.hpp"

namespace dgmg {

// Elements per block.  3D: the lines of one direction fill whole waves (P = 8: 243 of 256
// lanes; one element per block, 81 of 128, 32 instead of 22 us, two, 162 of 192, 27 us).
// 2D: about 256 nodes.
template <int NP, int DIM>
constexpr int apply_epb() {
  return DIM == 3 ? imax(1, (NP < 7 ? 128 : 256) / (NP * NP)) : imax(1, 256 / (NP * NP));
}
template <int NP, int DIM>
constexpr int apply_threads() {
  return DIM == 3 ? round64(apply_epb<NP, DIM>() * NP * NP) : imin(576, round64(apply_epb<NP, DIM>() * NP * NP));
}
// 3D: the neighbours along direction 0 outside the block are staged in the tile of
// contributions, left and right at once, or (one large element per block, where LDS
// bounds the blocks of a CU) one after the other.
template <int NP>
constexpr bool apply_two_halos() {
  return NP < 12;
}
template <class T, int DIM, int NP>
size_t apply_shmem(bool periodic0) {
  constexpr int EPB = apply_epb<NP, DIM>();
  if (DIM == 2) return (size_t)5 * EPB * NP * NP * sizeof(T);
  const int halos = apply_two_halos<NP>() ? (EPB > 1 && periodic0 ? 4 : 2) : 1;
  return (size_t)(EPB + imax(EPB, halos)) * ipow(NP, 3) * sizeof(T);
}
// Waves per SIMD that the registers have to leave room for (P = 16 FP64: two blocks of
// five waves fit the LDS, and with room for three the lines spilled: 53 instead of 42 us).
template <class T, int NP>
constexpr int apply_occupancy() {
  return sizeof(T) == 8 ? (NP <= 9 ? 4 : (NP <= 13 ? 3 : 2)) : (NP <= 9 ? 6 : 4);
}

template <class T>
struct ApplyArgs {
  const T* x = nullptr;
  const T* f = nullptr;
  T* y = nullptr;
  double* part = nullptr;
  const T* Ls = nullptr;
  const T* D = nullptr;
  const T* rho = nullptr;
  const T* J = nullptr;
  const T* ec[3] = {nullptr, nullptr, nullptr};  // ECOEF_N coefficients per element of a direction
  const int* active = nullptr;
  int n_elem = 0, nblk = 0;
  int N0 = 1, N1 = 1, N2 = 1;
  int per = 0;              // bit d: periodic in direction d
  uint32_t mg0 = 0, mg1 = 0;  // divisions by N0 and N1
};
template <class T>
ApplyArgs<T> apply_args(const LevelDev<T>& L, const T* x, const T* f, T* y, double* part, int nblk) {
  ApplyArgs<T> a;
  a.x = x;
  a.f = f;
  a.y = y;
  a.part = part;
  a.Ls = L.Ls;
  a.D = L.D;
  a.rho = L.rho;
  a.J = L.J;
  for (int d = 0; d < L.dim; ++d) {
    a.ec[d] = L.dir[d].ecoef;
    a.per |= L.dir[d].periodic ? 1 << d : 0;
  }
  a.active = L.active;
  a.n_elem = L.n_elem;
  a.nblk = nblk;
  a.N0 = L.dir[0].N;
  a.N1 = L.dir[1].N;
  a.N2 = L.dim == 3 ? L.dir[2].N : 1;
  a.mg0 = div_magic(L.n_elem, a.N0);
  a.mg1 = div_magic(L.n_elem, a.N1);
  return a;
}

// a b rounded by itself, not as a part of a fused multiply-add: each direction's
// contribution is a value of its own, the same wherever it is added up
template <class T>
__device__ __forceinline__ T mul_alone(T a, T b) {
#pragma clang fp contract(off)
  return a * b;
}

// BATCH: the arguments come from the work list bl (ntot logical blocks in all)
template <class T, int NP, int MODE, bool BATCH = false>
__global__ void __launch_bounds__((apply_threads<NP, 3>()))
    __attribute__((amdgpu_waves_per_eu((apply_occupancy<T, NP>()))))
    apply_kernel(ApplyArgs<T> a0, BatchList<ApplyArgs<T>> bl, int ntot) {
  constexpr int NE = NP * NP * NP, NLN = NP * NP, EPB = apply_epb<NP, 3>(), TH = apply_threads<NP, 3>();
  constexpr int P = NP - 1, NPC = (NP - 1) / 2 + 1;  // NPC: N_P of the next coarser level, P_c = floor(P / 2)
  constexpr bool TWO = apply_two_halos<NP>();
  static_assert(TWO || EPB == 1, "one halo at a time: one element per block");
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* sx = reinterpret_cast<T*>(smem_raw);  // the block's own elements
  T* tile = sx + EPB * NE;                 // contributions (first the halo elements of direction 0)
  __shared__ T sC[EPB * 3 * ECOEF_N];
  __shared__ T sJx[MODE == 3 ? NP * NPC : 1];
  __shared__ double red[16];
  __shared__ __align__(16) int sargs_raw[BATCH ? sizeof(ApplyArgs<T>) / sizeof(int) : 1];
  const ApplyArgs<T>* ap;
  int blk = 0;
  if constexpr (BATCH) {
    const int b = xcd_block(ntot);
    if (b < 0) return;
    ApplyArgs<T>* sargs = reinterpret_cast<ApplyArgs<T>*>(sargs_raw);
    blk = batch_pick(bl, b, sargs);
    ap = sargs;
  } else {
    ap = &a0;
  }
  // every argument into scalar registers by one group of loads
  const auto uni = [](int v) { return BATCH ? __builtin_amdgcn_readfirstlane(v) : v; };
  const auto ptr = [](auto* q) { return BATCH ? sgpr_ptr(q) : q; };
  const T *px = ptr(ap->x), *pf = ptr(ap->f), *pLs = ptr(ap->Ls), *pD = ptr(ap->D), *prho = ptr(ap->rho);
  const T *pe0 = ptr(ap->ec[0]), *pe1 = ptr(ap->ec[1]), *pe2 = ptr(ap->ec[2]);
  T* py = ptr(ap->y);
  const int* act = ptr(ap->active);
  int n_elem = uni(ap->n_elem), nblk = uni(ap->nblk), N0 = uni(ap->N0), N1 = uni(ap->N1), N2 = uni(ap->N2);
  int per = uni(ap->per);
  uint32_t mg0 = uni(ap->mg0), mg1 = uni(ap->mg1);
  if constexpr (!BATCH) {
    asm volatile("" : "+s"(px), "+s"(pf), "+s"(pLs), "+s"(pD), "+s"(prho), "+s"(pe0), "+s"(pe1), "+s"(pe2), "+s"(py),
                 "+s"(act), "+s"(n_elem), "+s"(nblk), "+s"(N0), "+s"(N1), "+s"(N2), "+s"(per), "+s"(mg0), "+s"(mg1));
    blk = xcd_block(nblk);
    if (blk < 0) return;
  }
  using G = const __attribute__((address_space(1))) T;   // global memory
  using CT = const __attribute__((address_space(4))) T;  // constant: scalar loads
  G *x = (G*)px, *f = (G*)pf, *rho = (G*)prho, *ec0 = (G*)pe0, *ec1 = (G*)pe1, *ec2 = (G*)pe2;
  auto* y = (__attribute__((address_space(1))) T*)py;
  CT *Ls = (CT*)pLs, *D0 = (CT*)pD, *DP = (CT*)(pD + P * NP);
  if (act != nullptr && *(const __attribute__((address_space(1))) int*)act == 0) return;
  const int e0 = uni(blk) * EPB, ne = imin(EPB, n_elem - e0), e_end = e0 + ne - 1;
  const int tid = threadIdx.x;
  const int64_t g0 = (int64_t)e0 * NE;
  G* xb = x + g0;
  const bool per0 = per & 1, per1 = per & 2, per2 = per & 4;

  // the own elements and the elements beside the block along direction 0: left of its first
  // and right of its last element; on a periodic row cut by the block also the other ends
  const int row0 = uni(div_by(e0, N0, mg0)) * N0, row1 = uni(div_by(e_end, N0, mg0)) * N0;
  const int hl = e0 > row0 ? e0 - 1 : (per0 ? row0 + N0 - 1 : e0);
  const int hr = e_end < row1 + N0 - 1 ? e_end + 1 : (per0 ? row1 : e_end);
  const int hl1 = row1 + N0 - 1, hr1 = row0;  // (used when per0 and the block spans rows)
  constexpr int CO = (EPB * NE + TH - 1) / TH, CH = (NE + TH - 1) / TH;
  T so[CO], sl[CH], sr[CH];
#pragma unroll
  for (int c = 0; c < CO; ++c) so[c] = xb[imin(tid + c * TH, ne * NE - 1)];
  auto load_halo = [&](T* s, int e) {
    G* xe = x + (int64_t)e * NE;
#pragma unroll
    for (int c = 0; c < CH; ++c) s[c] = xe[c + 1 < CH || NE % TH == 0 ? tid + c * TH : imin(tid + c * TH, NE - 1)];
  };
  auto store_halo = [&](const T* s, int slot) {
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int q = tid + c * TH;
      if (c + 1 < CH || NE % TH == 0 || q < NE) tile[slot * NE + q] = s[c];
    }
  };
  load_halo(sl, hl);
  load_halo(sr, hr);
  // coefficients of the block's elements
  for (int q = tid; q < ne * 3 * ECOEF_N; q += TH) {
    const int c = q % ECOEF_N, ed = q / ECOEF_N, el = ed / 3, d = ed - el * 3;
    const int e = e0 + el, r = div_by(e, N0, mg0), r2 = div_by(r, N1, mg1);
    G* ec = d == 0 ? ec0 + (e - r * N0) * ECOEF_N : (d == 1 ? ec1 + (r - r2 * N1) * ECOEF_N : ec2 + r2 * ECOEF_N);
    sC[q] = ec[c];
  }
  if constexpr (MODE == 3) {
    G* J = (G*)ptr(ap->J);
    for (int q = tid; q < NP * NPC; q += TH) sJx[q] = J[q];
  }
  // this thread's lines: element el, position (ia, ib) in the other directions, in order
  const bool has = tid < ne * NLN;
  const int el = has ? tid / NLN : 0, t = has ? tid - el * NLN : 0;
  const int ia = t % NP, ib = t / NP;
  const int e = e0 + el, rw = div_by(e, N0, mg0), m0 = e - rw * N0;
  const int m2 = div_by(rw, N1, mg1), m1 = rw - m2 * N1;
  const T ra = rho[ia], rb = rho[ib];
  // neighbours along d: m -/+ 1, wrapped when periodic, none (the element itself, masked) at a
  // Dirichlet end
  const bool l0 = m0 > 0 || per0, r0 = m0 < N0 - 1 || per0;
  const bool l1 = m1 > 0 || per1, r1 = m1 < N1 - 1 || per1;
  const bool l2 = m2 > 0 || per2, r2 = m2 < N2 - 1 || per2;
  const int st2 = N0 * N1;
  const int b1 = ia + ib * NP * NP;
  auto load_lines = [&](int nl, int nr, int base, auto stride, T* wl, T* wr) {
    G *pl = x + ((int64_t)nl * NE + base), *pr = x + ((int64_t)nr * NE + base);
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      wl[k] = pl[k * stride];
      wr[k] = pr[k * stride];
    }
  };
  using S0 = std::integral_constant<int, 1>;
  using S1 = std::integral_constant<int, NP>;
  using S2 = std::integral_constant<int, NP * NP>;
  T wl[NP], wr[NP];
  load_lines(m1 > 0 ? e - N0 : (per1 ? e + (N1 - 1) * N0 : e), m1 < N1 - 1 ? e + N0 : (per1 ? e - (N1 - 1) * N0 : e), b1,
             S1{}, wl, wr);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int c = 0; c < CO; ++c) {
    const int q = tid + c * TH;
    if (q < ne * NE) sx[q] = so[c];
  }
  store_halo(sl, 0);
  if constexpr (TWO) {
    store_halo(sr, 1);
    if constexpr (EPB > 1) {
      if (per0 && row1 != row0) {
        load_halo(sl, hl1);
        load_halo(sr, hr1);
        store_halo(sl, 2);
        store_halo(sr, 3);
      }
    }
  }
  __syncthreads();

  // The line's contribution mo * (L_d-row terms), row i handed to st(i, value).
  auto trace = [&](CT* row, const T* w, T& der) {
    der = 0;
#pragma unroll
    for (int k = 0; k < NP; ++k) der += row[k] * w[k];
  };
  auto line = [&](int d, const T* v, T dL, T uL, T dR, T uR, bool hasl, bool hasr, T mo, auto st) {
    const T* c = sC + (el * 3 + d) * ECOEF_N;
    T d0, dP;
    trace(D0, v, d0);
    trace(DP, v, dP);
    const T ml = hasl ? T(1) : T(0), mr = hasr ? T(1) : T(0);
    const T jl = v[0] - ml * uL, jr = v[P] - mr * uR;
    const T fl = c[E_CL] * d0 + c[E_CNL] * (ml * dL) + c[E_BL] * jl;
    const T fr = -c[E_CR] * dP - c[E_CNR] * (mr * dR) + c[E_BR] * jr;
    const T cl = c[E_CL] * jl, cr = c[E_CR] * jr, tdx = c[E_TWO_DX];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      T s = 0;
#pragma unroll
      for (int k = 0; k < NP; ++k) s += Ls[i * NP + k] * v[k];
      T o = tdx * s + cl * D0[i] - cr * DP[i];
      if (i == 0) o += fl;
      if (i == P) o += fr;
      st(i, mul_alone(mo, o));
    }
  };
  auto half = [&](int d) { return sC[(el * 3 + d) * ECOEF_N + E_HALF_DX]; };

  // ---- direction 0: neighbours in the block or in the halo slots
  {
    const int nl = m0 > 0 ? e - 1 : (per0 ? e + N0 - 1 : e), nr = m0 < N0 - 1 ? e + 1 : (per0 ? e - (N0 - 1) : e);
    const bool il = nl >= e0 && nl <= e_end, ir = nr >= e0 && nr <= e_end;
    const int ol = il ? (nl - e0) * NE : (EPB + (EPB == 1 || el == 0 ? 0 : 2)) * NE;
    const int orr = ir ? (nr - e0) * NE : (EPB + (TWO ? (EPB == 1 || el == ne - 1 ? 1 : 3) : 0)) * NE;
    T v[NP], dL, dR, uL, uR;
    const T* pv = sx + el * NE + t * NP;
#pragma unroll
    for (int k = 0; k < NP; ++k) v[k] = pv[k];
    {
      const T* p = sx + ol + t * NP;
      T w[NP];
#pragma unroll
      for (int k = 0; k < NP; ++k) w[k] = p[k];
      trace(DP, w, dL);
      uL = w[P];
    }
    if constexpr (!TWO) {
      __syncthreads();
      store_halo(sr, 0);
      __syncthreads();
    }
    {
      const T* p = sx + orr + t * NP;
      T w[NP];
#pragma unroll
      for (int k = 0; k < NP; ++k) w[k] = p[k];
      trace(D0, w, dR);
      uR = w[0];
    }
    __syncthreads();  // the halos are read, the tile may be written
    const T mo = half(1) * ra * half(2) * rb;
    T* o = tile + el * NE + t * NP;
    line(0, v, dL, uL, dR, uR, l0, r0, mo, [&](int i, T val) {
      if (has) o[i] = val;
    });
  }
  __syncthreads();

  // ---- direction 1; the next direction's lines are on the way meanwhile
  T dL, dR, uL, uR;
  trace(DP, wl, dL);
  trace(D0, wr, dR);
  uL = wl[P];
  uR = wr[0];
  load_lines(m2 > 0 ? e - st2 : (per2 ? e + (N2 - 1) * st2 : e), m2 < N2 - 1 ? e + st2 : (per2 ? e - (N2 - 1) * st2 : e),
             t, S2{}, wl, wr);
  __builtin_amdgcn_sched_barrier(0);
  {
    T v[NP];
    const T* pv = sx + el * NE + b1;
#pragma unroll
    for (int k = 0; k < NP; ++k) v[k] = pv[k * NP];
    const T mo = half(0) * ra * half(2) * rb;
    T* o = tile + el * NE + b1;
    line(1, v, dL, uL, dR, uR, l1, r1, mo, [&](int i, T val) {
      if (has) o[i * NP] += val;
    });
  }
  __syncthreads();

  // ---- direction 2 (f is not loaded before: its registers made FP64 lines spill)
  const int bz = el * NE + t;
  constexpr int SZ = NP * NP;
  T other[NP];
  if constexpr (MODE == 1 || MODE == 3) {
#pragma unroll
    for (int k = 0; k < NP; ++k) other[k] = (f + g0)[bz + k * SZ];
  }
  __builtin_amdgcn_sched_barrier(0);
  trace(DP, wl, dL);
  trace(D0, wr, dR);
  uL = wl[P];
  uR = wr[0];
  double acc = 0.0;
  {
    T v[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) v[k] = sx[bz + k * SZ];
    const T mo = half(0) * ra * half(1) * rb;
    const T* o = tile + bz;
    line(2, v, dL, uL, dR, uR, l2, r2, mo, [&](int i, T c) {
      const T val = o[i * SZ] + c;
      if (!has) return;
      if constexpr (MODE == 3) {
        sx[bz + i * SZ] = other[i] - val;  // (only this thread reads or writes the line now)
      } else {
        (y + g0)[bz + i * SZ] = MODE == 1 ? other[i] - val : val;
        if constexpr (MODE == 2) acc += (double)v[i] * (double)val;
      }
    });
  }
  if constexpr (MODE == 2) {
    const double s = block_sum(acc, red);
    if (tid == 0) ptr(ap->part)[blk] = s;
  }
  if constexpr (MODE == 3) {
    // the transfer kernel's restriction passes on the residual; y is the coarse vector
    constexpr int NEC = NPC * NPC * NPC;
    __syncthreads();
    xfer_pass<T, 3, NP, NPC, NE, 0, true, NPC>(sJx, sx, tile, ne);
    __syncthreads();
    xfer_pass<T, 3, NP, NPC, NE, 1, true, NPC>(sJx, tile, sx, ne);
    __syncthreads();
    xfer_pass<T, 3, NP, NPC, NE, 2, true, NPC>(sJx, sx, tile, ne);
    __syncthreads();
    for (int q = tid; q < ne * NEC; q += TH) {
      const int ec = q / NEC;
      (y + (int64_t)e0 * NEC)[q] = tile[ec * NE + q - ec * NEC];
    }
  }
}

// 2D grids that leave the GPU mostly idle, where the length of one thread's work is the
// time: a thread per node instead of one per line.  An element and
// its four neighbours come to LDS by coalesced loads, a thread per line and side takes the
// face terms (17 instead of 289 products in a row at P = 16), then every node adds up its
// two rows, matrix and values from LDS.
// Figures: apply_lines.
template <class T, int NP, int MODE, bool BATCH = false>
__global__ void __launch_bounds__((apply_threads<NP, 2>()))
    apply2_kernel(ApplyArgs<T> a0, BatchList<ApplyArgs<T>> bl, int ntot) {
  constexpr int NE = NP * NP, EPB = apply_epb<NP, 2>(), TH = apply_threads<NP, 2>();
  constexpr int P = NP - 1, NPC = (NP - 1) / 2 + 1, C = (EPB * NE + TH - 1) / TH;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* sx = reinterpret_cast<T*>(smem_raw);  // own elements, then left, right, below, above
  __shared__ T sLs[NP * NP], sD[2 * NP], srho[NP];
  __shared__ T sC[EPB * 2 * ECOEF_N];
  __shared__ T sF[EPB * 4 * NP * 2];
  __shared__ T sJx[MODE == 3 ? NP * NPC : 1];
  __shared__ double red[16];
  __shared__ __align__(16) int sargs_raw[BATCH ? sizeof(ApplyArgs<T>) / sizeof(int) : 1];
  const ApplyArgs<T>* ap;
  int blk = 0;
  if constexpr (BATCH) {
    const int b = xcd_block(ntot);
    if (b < 0) return;
    ApplyArgs<T>* sargs = reinterpret_cast<ApplyArgs<T>*>(sargs_raw);
    blk = batch_pick(bl, b, sargs);
    ap = sargs;
  } else {
    ap = &a0;
  }
  // every argument into scalar registers by one group of loads
  const auto uni = [](int v) { return BATCH ? __builtin_amdgcn_readfirstlane(v) : v; };
  const auto ptr = [](auto* q) { return BATCH ? sgpr_ptr(q) : q; };
  const T *px = ptr(ap->x), *pf = ptr(ap->f), *pLs = ptr(ap->Ls), *pD = ptr(ap->D), *prho = ptr(ap->rho);
  const T *pe0 = ptr(ap->ec[0]), *pe1 = ptr(ap->ec[1]), *pJ = ptr(ap->J);
  T* py = ptr(ap->y);
  const int* act = ptr(ap->active);
  int n_elem = uni(ap->n_elem), nblk = uni(ap->nblk), N0 = uni(ap->N0), N1 = uni(ap->N1), per = uni(ap->per);
  uint32_t mg0 = uni(ap->mg0);
  if constexpr (!BATCH) {
    asm volatile("" : "+s"(px), "+s"(pf), "+s"(pLs), "+s"(pD), "+s"(prho), "+s"(pe0), "+s"(pe1), "+s"(pJ), "+s"(py),
                 "+s"(act), "+s"(n_elem), "+s"(nblk), "+s"(N0), "+s"(N1), "+s"(per), "+s"(mg0));
    blk = xcd_block(nblk);
    if (blk < 0) return;
  }
  using G = const __attribute__((address_space(1))) T;  // global memory
  G *x = (G*)px, *f = (G*)pf, *ec0 = (G*)pe0, *ec1 = (G*)pe1, *gLs = (G*)pLs, *gD = (G*)pD, *grho = (G*)prho;
  auto* y = (__attribute__((address_space(1))) T*)py;
  if (act != nullptr && *(const __attribute__((address_space(1))) int*)act == 0) return;
  const int e0 = uni(blk) * EPB, ne = imin(EPB, n_elem - e0), n = ne * NE;
  const int tid = threadIdx.x;
  const int64_t g0 = (int64_t)e0 * NE;
  const bool per0 = per & 1, per1 = per & 2;
  T so[C], sn[4][C], other[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int q = imin(tid + c * TH, n - 1), el = q / NE, l = q - el * NE;
    const int e = e0 + el, m1 = div_by(e, N0, mg0), m0 = e - m1 * N0;
    // neighbours: m -/+ 1, wrapped when periodic, the element itself (masked) at a Dirichlet end
    const int nb[4] = {m0 > 0 ? e - 1 : (per0 ? e + N0 - 1 : e), m0 < N0 - 1 ? e + 1 : (per0 ? e - (N0 - 1) : e),
                       m1 > 0 ? e - N0 : (per1 ? e + (N1 - 1) * N0 : e),
                       m1 < N1 - 1 ? e + N0 : (per1 ? e - (N1 - 1) * N0 : e)};
    so[c] = x[g0 + q];
#pragma unroll
    for (int s = 0; s < 4; ++s) sn[s][c] = x[(int64_t)nb[s] * NE + l];
    if constexpr (MODE == 1 || MODE == 3) other[c] = f[g0 + q];
  }
  for (int q = tid; q < NP * NP; q += TH) sLs[q] = gLs[q];
  for (int q = tid; q < 2 * NP; q += TH) sD[q] = gD[q < NP ? q : P * NP + q - NP];
  for (int q = tid; q < NP; q += TH) srho[q] = grho[q];
  if constexpr (MODE == 3) {
    G* J = (G*)pJ;
    for (int q = tid; q < NP * NPC; q += TH) sJx[q] = J[q];
  }
  for (int q = tid; q < ne * 2 * ECOEF_N; q += TH) {
    const int c = q % ECOEF_N, ed = q / ECOEF_N, e = e0 + ed / 2, m1 = div_by(e, N0, mg0);
    sC[q] = ed & 1 ? ec1[m1 * ECOEF_N + c] : ec0[(e - m1 * N0) * ECOEF_N + c];
  }
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int q = tid + c * TH;
    if (q >= n) continue;
    sx[q] = so[c];
#pragma unroll
    for (int s = 0; s < 4; ++s) sx[(s + 1) * EPB * NE + q] = sn[s][c];
  }
  __syncthreads();
  // face terms of line ln of element el along direction d at its left (right) end: the
  // flux and the jump's weight
  for (int q = tid; q < ne * 4 * NP; q += TH) {
    const int el = q / (4 * NP), s = q / NP % 4, ln = q % NP, d = s >> 1, right = s & 1;
    const int e = e0 + el, m1 = div_by(e, N0, mg0), m = d ? m1 : e - m1 * N0;
    const T mask = (d ? per1 : per0) || (right ? m < (d ? N1 : N0) - 1 : m > 0) ? T(1) : T(0);
    const int base = el * NE + (d ? ln : ln * NP), st = d ? NP : 1;
    const T *v = sx + base, *w = sx + (s + 1) * EPB * NE + base;
    const T *Dv = sD + (right ? NP : 0), *Dw = sD + (right ? 0 : NP);
    T dv = 0, dw = 0;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      dv += Dv[k] * v[k * st];
      dw += Dw[k] * w[k * st];
    }
    const T* c = sC + (el * 2 + d) * ECOEF_N;
    const T j = v[right ? P * st : 0] - mask * w[right ? 0 : P * st];
    const T cj = c[right ? E_CR : E_CL], cn = c[right ? E_CNR : E_CNL], cb = c[right ? E_BR : E_BL];
    const T sg = right ? T(-1) : T(1);
    sF[2 * q] = sg * cj * dv + sg * cn * (mask * dw) + cb * j;
    sF[2 * q + 1] = sg * (cj * j);
  }
  __syncthreads();
  double acc = 0.0;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int q = tid + c * TH;
    if (q >= n) continue;
    const int el = q / NE, l = q - el * NE, i1 = l / NP, i0 = l - i1 * NP;
    const T* u = sx + el * NE;
    const T *c0 = sC + el * 2 * ECOEF_N, *c1 = c0 + ECOEF_N;
    const T *f0 = sF + 2 * (el * 4 * NP + i1), *f1 = sF + 2 * (el * 4 * NP + 2 * NP + i0);
    T s0 = 0, s1 = 0;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      s0 += sLs[i0 * NP + k] * u[i1 * NP + k];
      s1 += sLs[i1 * NP + k] * u[k * NP + i0];
    }
    T o0 = c0[E_TWO_DX] * s0 + f0[1] * sD[i0] + f0[2 * NP + 1] * sD[NP + i0];
    T o1 = c1[E_TWO_DX] * s1 + f1[1] * sD[i1] + f1[2 * NP + 1] * sD[NP + i1];
    if (i0 == 0) o0 += f0[0];
    if (i0 == P) o0 += f0[2 * NP];
    if (i1 == 0) o1 += f1[0];
    if (i1 == P) o1 += f1[2 * NP];
    const T val = mul_alone(c1[E_HALF_DX] * srho[i1], o0) + mul_alone(c0[E_HALF_DX] * srho[i0], o1);
    if constexpr (MODE == 3) {
      sx[EPB * NE + q] = other[c] - val;  // (the neighbours are no longer needed)
    } else {
      (y + g0)[q] = MODE == 1 ? other[c] - val : val;
      if constexpr (MODE == 2) acc += (double)u[l] * (double)val;
    }
  }
  if constexpr (MODE == 2) {
    const double s = block_sum(acc, red);
    if (tid == 0) ptr(ap->part)[blk] = s;
  }
  if constexpr (MODE == 3) {
    // the transfer kernel's restriction passes on the residual; y is the coarse vector
    constexpr int NEC = NPC * NPC;
    T *r = sx + EPB * NE, *b = r + EPB * NE, *o = b + EPB * NE;
    __syncthreads();
    xfer_pass<T, 2, NP, NPC, NE, 0, true, NPC>(sJx, r, b, ne);
    __syncthreads();
    xfer_pass<T, 2, NP, NPC, NE, 1, true, NPC>(sJx, b, o, ne);
    __syncthreads();
    for (int q = tid; q < ne * NEC; q += TH) {
      const int ec = q / NEC;
      (y + (int64_t)e0 * NEC)[q] = o[ec * NE + q - ec * NEC];
    }
  }
}

// The form for 2D grids that fill the GPU and for 3D grids that leave it mostly idle: a
// thread per line of one element in one direction, the lines of all directions at once
// (their loads overlap instead of forming one chain per direction), one LDS tile of
// contributions per direction.
// Elements per block: lines of all directions fill about 256 threads.
template <int NP, int DIM>
constexpr int lines_epb() {
  return imax(1, 256 / (DIM * ipow(NP, DIM - 1)));
}
template <int NP, int DIM>
constexpr int lines_threads() {
  return imin(1024, round64(lines_epb<NP, DIM>() * DIM * ipow(NP, DIM - 1)));
}
// Own elements staged in LDS (coalesced loads) when the tiles are small: the
// lines of the block's own elements are then read from LDS and only the
// neighbours' lines from global memory.  A line along direction 0 is contiguous,
// so the lanes of a wave (one line each) are NP values apart and a load touches
// about one cache line per lane: staging removes the costliest third of the line
// loads.
template <int NP, int DIM>
constexpr bool lines_stage_own() {
  return NP <= 9 && lines_epb<NP, DIM>() * DIM * ipow(NP, DIM - 1) <= 1024;
}
template <class T, int DIM, int NP>
constexpr size_t lines_shmem() {
  return (size_t)(DIM + (lines_stage_own<NP, DIM>() ? 1 : 0)) * lines_epb<NP, DIM>() * ipow(NP, DIM) * sizeof(T);
}

// Everything one line needs besides its own values: indices, the neighbours'
// lines (masks ml, mr), the face coefficients and the mass factor.
template <class T, int NP>
struct ApplyLine {
  int d, el, base, stride;
  T ml, mr, mo;
  T c_two_dx, c_cl, c_cnl, c_bl, c_cr, c_cnr, c_br;
  T wlv[NP], wrv[NP];
};

// BATCH: the arguments come from the work list bl (ntot logical blocks in all)
template <class T, int DIM, int NP, int MODE, bool BATCH = false>
__global__ void __launch_bounds__(1024) apply_lines_kernel(ApplyArgs<T> a0, BatchList<ApplyArgs<T>> bl, int ntot) {
  constexpr int NE = ipow(NP, DIM), NLN = ipow(NP, DIM - 1), EPB = lines_epb<NP, DIM>();
  constexpr int P = NP - 1;
  constexpr bool STAGE = lines_stage_own<NP, DIM>();
  extern __shared__ __align__(16) unsigned char smem_raw[];
  // per-direction contribution tiles, then (STAGE) the block's own elements
  T* sy = reinterpret_cast<T*>(smem_raw);
  T* sx = sy + DIM * EPB * NE;
  __shared__ double red[16];
  __shared__ __align__(16) int sargs_raw[BATCH ? sizeof(ApplyArgs<T>) / sizeof(int) : 1];
  ApplyArgs<T>* sargs = reinterpret_cast<ApplyArgs<T>*>(sargs_raw);
  const ApplyArgs<T>* ap;
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
  const T* __restrict__ x = ap->x;
  const T* __restrict__ f = ap->f;
  T* __restrict__ y = ap->y;
  double* __restrict__ part = ap->part;
  if (inactive(ap->active)) return;
  const int e0 = blk * EPB;
  const int ne = imin(EPB, ap->n_elem - e0);
  const int tid = threadIdx.x, nth = blockDim.x;
  const int64_t g0 = (int64_t)e0 * NE;
  const int N1 = ap->N0, N2 = ap->N1;
  // stiffness matrix rows: uniform addresses in the constant address space,
  // so the row loop reads them with scalar loads into SGPR operands; rows
  // longer than 72 bytes (2D, large P) would not fit the scalar registers and
  // are staged in LDS instead (uniform-address reads)
  constexpr bool SLS = NP * sizeof(T) <= 72;
  __shared__ T sLsL[SLS ? 1 : NP * NP];
  if constexpr (!SLS) {
    for (int q = tid; q < NP * NP; q += nth) sLsL[q] = ap->Ls[q];
    __syncthreads();
  }
  // MODE 3: the interpolation matrix J (NP x NPC, row-major) of the restriction
  constexpr int NPC = (NP - 1) / 2 + 1;  // N_P of the next coarser level, P_c = floor(P / 2)
  static_assert(MODE != 3 || STAGE, "the fused restriction needs the own-element LDS buffer");
  __shared__ T sJx[MODE == 3 ? NP * NPC : 1];
  if constexpr (MODE == 3)
    for (int q = tid; q < NP * NPC; q += nth) sJx[q] = ap->J[q];
  using CT = const __attribute__((address_space(4))) T;
  CT* __restrict__ Ls = (CT*)ap->Ls;
  CT* __restrict__ D0 = (CT*)ap->D;
  CT* __restrict__ DP = (CT*)(ap->D + P * NP);
  const T* __restrict__ rho = ap->rho;
  const int per_dir = ne * NLN;
  // per-direction kernel arguments in scalar registers; the per-lane choice
  // below is arithmetic with 0/1 flags (a select chain over them gets turned
  // into a small scratch array or into per-lane loads of the arguments)
  using GT = const __attribute__((address_space(1))) T;  // global memory
  GT* ec0 = (GT*)sgpr_ptr(ap->ec[0]);
  GT* ec1 = (GT*)sgpr_ptr(ap->ec[1]);
  GT* ec2 = (GT*)sgpr_ptr(ap->ec[DIM - 1]);
  const int64_t eo1 = ec1 - ec0, eo2 = ec2 - ec0;
  const int per0 = __builtin_amdgcn_readfirstlane(ap->per & 1);
  const int per1 = __builtin_amdgcn_readfirstlane(ap->per & 2);
  const int per2 = __builtin_amdgcn_readfirstlane(ap->per & (1 << (DIM - 1)));
  const int N3 = __builtin_amdgcn_readfirstlane(DIM == 3 ? ap->N2 : ap->N1);
  // The vector the epilogue reads besides the tiles (f for the residual, x for
  // the dot product) is fetched now, so that its latency overlaps the line work
  // (launches use lines_threads() threads, so FQ values per thread cover the block).
  constexpr int TH = lines_threads<NP, DIM>(), FQ = (EPB * NE + TH - 1) / TH;
  constexpr bool PREF = MODE != 0 && NP <= 9;
  T pre[PREF ? FQ : 1];
  if constexpr (PREF) {
    const T* __restrict__ src = (MODE == 1 || MODE == 3) ? f : x;
#pragma unroll
    for (int j = 0; j < FQ; ++j) {
      const int q = tid + j * nth;
      pre[j] = q < ne * NE ? src[g0 + q] : T(0);
    }
  }
  // Loads of line q (all issued as one group): neighbours' lines (unconditional
  // loads at a valid address, masked later), coefficients, mass factors and,
  // unless staged, the own line into v.
  auto prep = [&](int q, ApplyLine<T, NP>& A, T* v, bool own) {
    const int d = q / per_dir;
    const int ln = q - d * per_dir;
    const int el = ln / NLN, t = ln - el * NLN;
    const int e = e0 + el;
    int m[3];
    m[0] = e % N1;
    m[1] = DIM == 3 ? (e / N1) % N2 : e / N1;
    m[2] = DIM == 3 ? e / (N1 * N2) : 0;
    // per-direction fields chosen per lane (the direction varies inside a wave)
    const int f0 = d == 0, f1 = d == 1, f2 = d == 2;
    const int md = f0 * m[0] + f1 * m[1] + f2 * m[2];
    const int Nd = f0 * N1 + f1 * N2 + f2 * N3;
    const int perd = f0 * per0 + f1 * per1 + f2 * per2;
    GT* __restrict__ ecoef = ec0 + (f1 * eo1 + f2 * eo2);
    const int estride = f0 + f1 * N1 + f2 * (N1 * N2);
    // line base and stride inside the element; indices of the other directions
    const int ia = t % NP, ib = t / NP;  // local indices of the other directions (in order)
    int base, stride;
    if (d == 0) {
      base = t * NP; stride = 1;
    } else if (d == 1) {
      base = ia + ib * NP * NP; stride = NP;
    } else {
      base = t; stride = NP * NP;
    }
    A.d = d;
    A.el = el;
    A.base = base;
    A.stride = stride;
    // neighbours along d: m -/+ 1, wrapped when periodic, none (-1) at a
    // Dirichlet end (the element neighbour table of the setup, computed here so
    // that no load depends on another)
    const int nl = md > 0 ? md - 1 : (perd ? Nd - 1 : -1);
    const int nr = md < Nd - 1 ? md + 1 : (perd ? 0 : -1);
    A.ml = nl >= 0 ? T(1) : T(0);
    A.mr = nr >= 0 ? T(1) : T(0);
    if (own) {
#pragma unroll
      for (int k = 0; k < NP; ++k) v[k] = x[g0 + el * NE + base + k * stride];
    }
    GT* c = ecoef + md * ECOEF_N;
    A.c_two_dx = c[E_TWO_DX];
    A.c_cl = c[E_CL];
    A.c_cnl = c[E_CNL];
    A.c_bl = c[E_BL];
    A.c_cr = c[E_CR];
    A.c_cnr = c[E_CNR];
    A.c_br = c[E_BR];
    const T ra = rho[ia], rb = DIM == 3 ? rho[ib] : T(1);
    T ha, hb;  // half element sizes of the other directions
    if (DIM == 2) {
      ha = d == 0 ? ec1[m[1] * ECOEF_N + E_HALF_DX] : ec0[m[0] * ECOEF_N + E_HALF_DX];
      hb = T(1);
    } else {
      const T h0 = ec0[m[0] * ECOEF_N + E_HALF_DX];
      const T h1 = ec1[m[1] * ECOEF_N + E_HALF_DX];
      const T h2 = ec2[m[2] * ECOEF_N + E_HALF_DX];
      ha = d == 0 ? h1 : h0;
      hb = d == 2 ? h1 : h2;
    }
    // mass factor of the other directions at this line
    A.mo = DIM == 2 ? ha * ra : ha * ra * hb * rb;
    const T* wl = x + (int64_t)(e + (nl >= 0 ? nl - md : 0) * estride) * NE + base;
    const T* wr = x + (int64_t)(e + (nr >= 0 ? nr - md : 0) * estride) * NE + base;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      A.wlv[k] = wl[k * stride];
      A.wrv[k] = wr[k * stride];
    }
  };
  // the line's contribution mo * (L_d-row terms) into its direction's tile
  auto finish = [&](const ApplyLine<T, NP>& A, const T* v) {
    T d0 = 0, dP = 0, dL = 0, dR = 0;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      d0 += D0[k] * v[k];
      dP += DP[k] * v[k];
      dL += DP[k] * A.wlv[k];
      dR += D0[k] * A.wrv[k];
    }
    const T uL = A.ml * A.wlv[P], uR = A.mr * A.wrv[0];
    dL *= A.ml;
    dR *= A.mr;
    const T jl = v[0] - uL, jr = v[P] - uR;
    const T fl = A.c_cl * d0 + A.c_cnl * dL + A.c_bl * jl;
    const T fr = -A.c_cr * dP - A.c_cnr * dR + A.c_br * jr;
    const T cl = A.c_cl * jl, cr = A.c_cr * jr, tdx = A.c_two_dx;
    T* __restrict__ syd = sy + (A.d * ne + A.el) * NE + A.base;
#pragma unroll 1  // one row of Ls live at a time (registers for the line data)
    for (int i = 0; i < NP; ++i) {
      T s = 0;
#pragma unroll
      for (int k = 0; k < NP; ++k) {
        if constexpr (SLS) s += Ls[__builtin_amdgcn_readfirstlane(i) * NP + k] * v[k];
        else s += sLsL[i * NP + k] * v[k];
      }
      const int iu = __builtin_amdgcn_readfirstlane(i);
      T o = tdx * s + cl * D0[iu] - cr * DP[iu];
      if (i == 0) o += fl;
      if (i == P) o += fr;
      syd[i * A.stride] = A.mo * o;
    }
  };
  if constexpr (STAGE) {
    // one line per thread (the launch covers all lines of the block)
    constexpr int SQ = (EPB * NE + TH - 1) / TH;
    T st[SQ];
#pragma unroll
    for (int j = 0; j < SQ; ++j) {
      const int q = tid + j * nth;
      st[j] = q < ne * NE ? x[g0 + q] : T(0);
    }
    const bool has = tid < DIM * per_dir;
    ApplyLine<T, NP> A;
    T v[NP];
    prep(has ? tid : 0, A, v, false);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < SQ; ++j) {
      const int q = tid + j * nth;
      if (q < ne * NE) sx[q] = st[j];
    }
    __syncthreads();
    if (has) {
#pragma unroll
      for (int k = 0; k < NP; ++k) v[k] = sx[A.el * NE + A.base + k * A.stride];
      finish(A, v);
    }
  } else {
    for (int q = tid; q < DIM * per_dir; q += nth) {
      ApplyLine<T, NP> A;
      T v[NP];
      prep(q, A, v, true);
      if constexpr (NP <= 9) __builtin_amdgcn_sched_barrier(0);
      finish(A, v);
    }
  }
  __syncthreads();
  double acc = 0.0;
  const int dstride = ne * NE;
  auto out = [&](int q, T other) {
    T val = sy[q] + sy[dstride + q];
    if (DIM == 3) val += sy[2 * dstride + q];
    if (MODE == 0) {
      y[g0 + q] = val;
    } else if (MODE == 1) {
      y[g0 + q] = other - val;
    } else if (MODE == 3) {
      sx[q] = other - val;  // the own elements' x are no longer needed
    } else {
      y[g0 + q] = val;
      acc += (double)other * (double)val;
    }
  };
  if constexpr (PREF) {
#pragma unroll
    for (int j = 0; j < FQ; ++j) {
      const int q = tid + j * nth;
      if (q < ne * NE) out(q, pre[j]);
    }
  } else if constexpr (MODE == 0) {
    for (int q = tid; q < ne * NE; q += nth) out(q, T(0));
  } else {
    // every load of f (x) issued before the sums that use them
    const T* __restrict__ src = (MODE == 1 || MODE == 3) ? f : x;
    staged_copy<T, TH, EPB * NE>([&](int q) { return src[g0 + q]; }, [&](int q, T v) { out(q, v); }, ne * NE);
  }
  if (MODE == 2) {
    const double s = block_sum(acc, red);
    if (tid == 0) part[blk] = s;
  }
  if constexpr (MODE == 3) {
    // the transfer kernel's restriction passes, on the residual in LDS (the
    // direction tiles serve as the two pass buffers); y is the coarse vector
    constexpr int NEC = ipow(NPC, DIM);
    __syncthreads();
    T* bA = sy;
    T* bB = sy + EPB * NE;
    xfer_pass<T, DIM, NP, NPC, NE, 0, true, NPC>(sJx, sx, bA, ne);
    __syncthreads();
    xfer_pass<T, DIM, NP, NPC, NE, 1, true, NPC>(sJx, bA, bB, ne);
    __syncthreads();
    const T* res = bB;
    if constexpr (DIM == 3) {
      xfer_pass<T, DIM, NP, NPC, NE, 2, true, NPC>(sJx, bB, bA, ne);
      __syncthreads();
      res = bA;
    }
    T* yc = y + (int64_t)e0 * NEC;
    for (int q = tid; q < ne * NEC; q += nth) {
      const int el = q / NEC;
      yc[q] = res[el * NE + q - el * NEC];
    }
  }
}

// The form of a grid's apply (of the grid, also when grids share a launch, so that a batch
// gives what its grids give alone).  2D: a thread per node up to 1.5 MB of level vector,
// where the line form's chain of products is the time (residual of 16x16 P = 16 FP64 11.8
// against 4.9 us); beyond, its LDS reads bind it (128x128 P = 16 FP64 199 against 60 us; the two
// meet at 200000 to 300000 nodes in FP64, twice that in FP32).  P <= 2: lines (3.6 against
// 4.0 us).  3D, P <= 8: lines while the directions in turn are the longer chain, up to
// 1 MB in FP32, 1.25 MB in FP64, 1.75 MB (P = 6) and 3 MB (P = 8).  Residual, lines / in turn,
// us: FP64 P = 3 13^3 4.7 / 5.3, P = 6 8^3 5.4 / 6.2, P = 8 6^3 5.9 / 7.3, 8^3 6.9 / 7.7; beyond the
// lines (these in their form before, 0.3 us slower) P = 4 12^3 6.0 / 5.3, P = 6 10^3 7.3 / 6.3,
// P = 8 10^3 9.8 / 9.8, 12^3 14.8 / 12.2, FP32 P = 4 13^3 5.5 / 4.8, P = 8 8^3 6.6 / 6.4.
template <class T, int DIM, int NP>
constexpr bool apply_lines(int n_elem) {
  const int64_t bytes = (int64_t)n_elem * ipow(NP, DIM) * (int64_t)sizeof(T);
  if (DIM == 2) return NP <= 3 || bytes > (3 << 19);
  return NP <= 9 && bytes <= (sizeof(T) == 4 ? 1 << 20 : (NP == 9 ? 3 << 20 : (NP == 7 ? 7 << 18 : 5 << 18)));
}
template <int DIM, int NP>
constexpr bool apply_lines_built() {
  return DIM == 2 || NP <= 9;
}

template <class T, int DIM, int NP, int MODE, bool BATCH>
void apply_go(const ApplyArgs<T>& a, const BatchList<ApplyArgs<T>>& bl, int nlog, bool lines, hipStream_t s) {
  const auto go = [&](auto kernel, int th, size_t shm) {
    if (shm > 65536)
      (void)hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
    hipLaunchKernelGGL(kernel, dim3(xcd_grid(nlog)), dim3(th), shm, s, a, bl, nlog);
  };
  if constexpr (apply_lines_built<DIM, NP>() && (MODE != 3 || lines_stage_own<NP, DIM>())) {
    if (lines)
      return go(apply_lines_kernel<T, DIM, NP, MODE, BATCH>, lines_threads<NP, DIM>(), lines_shmem<T, DIM, NP>());
  }
  const size_t shm = apply_shmem<T, DIM, NP>(BATCH || (a.per & 1));
  if constexpr (DIM == 3) go(apply_kernel<T, NP, MODE, BATCH>, apply_threads<NP, DIM>(), shm);
  else if constexpr (NP > 3) go(apply2_kernel<T, NP, MODE, BATCH>, apply_threads<NP, DIM>(), shm);
}

// Blocks of one grid's apply.
template <class T, int DIM, int NP>
int apply_blocks(int n_elem) {
  const int epb = apply_lines<T, DIM, NP>(n_elem) ? lines_epb<NP, DIM>() : apply_epb<NP, DIM>();
  return (n_elem + epb - 1) / epb;
}

// The fused residual + restriction (mode 3) is built for coarse levels whose order follows
// P_c = floor(P / 2), in the line form where it stages the own elements in LDS.
template <class T, int DIM, int NP>
bool apply_mode3_ok(const LevelDev<T>& L) {
  return !(DIM == 3 && NP > 17) && L.NPc == (NP - 1) / 2 + 1 && L.J != nullptr &&
         (!apply_lines<T, DIM, NP>(L.n_elem) || lines_stage_own<NP, DIM>());
}

template <class T, int DIM, int NP, bool BATCH>
int apply_mode(int mode, const ApplyArgs<T>& a, const BatchList<ApplyArgs<T>>& bl, int nlog, bool lines, hipStream_t s) {
  if (mode == 0) apply_go<T, DIM, NP, 0, BATCH>(a, bl, nlog, lines, s);
  else if (mode == 1) apply_go<T, DIM, NP, 1, BATCH>(a, bl, nlog, lines, s);
  else if (mode == 2) apply_go<T, DIM, NP, 2, BATCH>(a, bl, nlog, lines, s);
  else if (lines && !lines_stage_own<NP, DIM>()) return -4;
  else apply_go<T, DIM, NP, 3, BATCH>(a, bl, nlog, lines, s);
  return 0;
}

template <class T, int DIM, int NP>
int apply_launch(const LevelDev<T>& L, int mode, const T* x, const T* f, T* y, double* part,
                 int* nblk_out, hipStream_t s) {
  const int nblk = apply_blocks<T, DIM, NP>(L.n_elem);
  if (nblk_out) *nblk_out = nblk;
  // fused residual + restriction: otherwise the caller runs the two steps
  if (mode == 3 && !apply_mode3_ok<T, DIM, NP>(L)) return -4;
  return apply_mode<T, DIM, NP, false>(mode, apply_args(L, x, f, y, part, nblk), BatchList<ApplyArgs<T>>{}, nblk,
                                       apply_lines<T, DIM, NP>(L.n_elem), s);
}

// One launch over the applies of many grids (same NP, mode and form): ntot logical
// blocks, grid g's apply_blocks in the range of bl.
template <class T, int DIM, int NP>
int apply_batch_launch(int mode, bool lines, const BatchList<ApplyArgs<T>>& bl, int ntot, hipStream_t s) {
  return apply_mode<T, DIM, NP, true>(mode, ApplyArgs<T>{}, bl, ntot, lines, s);
}

}  // namespace dgmg
