// The RK stage from face traces (multi-step calls and batches, the FP64, FP64
// perturbation and FP32 perturbation forms).
//
// A face node's viscous flux and diffusion norm ||n^T G n||_2 need the
// neighbour's gradient there.  The stage kernel of a single right-hand side
// (kernels.hip) rebuilds it from the neighbour's 4 Np nodal values for every
// face, on both sides.  Between the stages of a step nothing forces that:
// the element that has just computed its new state can form its own gradient,
// viscous normal flux and norm once, and leave four numbers per face node --
//   (vn_1, vn_2, vn_3, largest norm of the face)      (vn_0 is zero)
// -- for the next stage, where each side reads its own and the neighbour's.
// The neighbour's normal is the own one negated exactly, and the matrix-core
// gradient equals the vector unit's fused multiply-add chain bit for bit, so
// both forms of the stage give the same bits (checked in the tests).
//
// Per element this writes and reads 96 (p + 1) bytes of traces in FP64 (48 in
// FP32) and forms the gradient once more on the matrix cores; it saves the
// neighbour's block (4 Np values), 16 Np flops per face node and one of the
// two norms and viscous fluxes, and with the blocks gone from LDS and the
// vector unit no longer reading the operator fragments at per-lane addresses,
// FP64 at p >= 5 runs two waves per SIMD instead of one.
//
// Measured against the stage from the neighbours' states, us a stage on 20,480
// elements (in brackets 327,680): p = 1 FP64 18.2 -> 15.1 (255 -> 137), p = 2 FP64
// 20.6 -> 17.9 (286 -> 191), p = 4 FP32 18.5 -> 15.9 (228 -> 203) and FP64 25.7 ->
// 22.1, p = 5 FP32 39 -> 28, p = 6 FP32 37 -> 31.6 and FP64 73 -> 50.  What bounds
// it: on 20,480 elements the issue and latency of a few waves per SIMD (p = 4 FP32:
// 870 vector and 36 matrix instructions a tile, five tiles a SIMD; a wave waits
// for memory, LDS or its turn in two thirds of its cycles) after a launch's cold first
// loads; beyond the last-level cache memory (p = 4 FP32: 0.95 GB a stage at 4.5
// TB/s, 92 % of a large copy's rate).
#pragma once

#include <hip/hip_runtime.h>

#include "stage_device.h"

namespace dgmi {

template <int N, typename T, bool LARGE = false>
struct TraceOrder {
  using O = Order<N, T>;
  static constexpr int Np = O::Np, Nfp = O::Nfp, NF = O::NF, S = O::S, NT = O::NT, KS = O::KS,
                       KF = O::KF, RS = O::RS, HRS = O::HRS, ROWC = O::ROWC, ROWE = O::ROWE;
  static constexpr int EPT = trace_elements_per_tile(N, LARGE);
  static constexpr int G = (EPT + 3) / 4;  // groups of four element slots (16 matrix-core rows)
  // Where one 16-column tile and one row group hold the elements (p = 3, 4) a
  // lane updates the outputs that the matrix cores leave in it; elsewhere that
  // layout fills 24 to 48 of the 64 lanes in each of several passes, so the
  // residual goes through LDS and a lane takes values lane + 64 q of the
  // tile's run of EPT element blocks (p = 1: 2 values instead of 12, p = 5:
  // 4 instead of 8).  The tile's states are loaded the same way.  On a mesh beyond the
  // last-level cache (LARGE) every order does (whole cache lines).
  static constexpr bool FLAT = G * NT > 1 || LARGE;
  static constexpr int BE = FLAT ? EPT : 1, EB = EPT / BE;
  static constexpr int NQ = (BE * S + 63) / 64;
  static constexpr int NG = (EPT * kGeoStride + 63) / 64;
  // the volume flux in one pass over (element, node) pairs packed onto the
  // lanes where the matrix-core layout would need several
  static constexpr bool PACK = EPT * Np <= 64 && G * NT > 1;
  // per-wave LDS (elements of T): state rows, flux rows F_r | F_s; the face
  // terms h | qr | qs follow the divergence, which has read the flux rows by
  // then, so they take the flux area; in FP64 at p >= 5 the state rows too
  // (the stage re-reads K0), which lets two workgroups share a CU's LDS
  static constexpr int U_SZ = G * 16 * RS, F_SZ = G * 32 * RS, H_SZ = G * 48 * HRS;
  static constexpr bool OVER = sizeof(T) == 8 && N >= 5;
  static constexpr int H_OFF = OVER ? 0 : U_SZ;
  static constexpr int AREA = U_SZ + F_SZ > H_OFF + H_SZ ? U_SZ + F_SZ : H_OFF + H_SZ;
  static constexpr int WAVE_SZ = (AREA + EPT * kGeoStride + 3) / 4 * 4;
  static_assert(!FLAT || G * 16 * RS <= H_SZ, "the residual rows take the face terms' area");
  static constexpr int PAD = 4 * KS - Np;  // pad columns that the products over the nodes read
  static constexpr int WAVES = 4;
  // registers: three waves per SIMD in FP32, two in FP64 (four and three spill:
  // p = 4 FP32 16.4 -> 18.1 us, FP64 22.6 -> 24.6).  K1 / K0 are loaded before the
  // face pass where they fit beside it (p <= 4; after it, p = 2 FP64 on 20,480
  // elements 17.6 -> 17.9); at p = 5 in FP32 they spill there (28 -> 35 us).  The
  // next tile's own data come after the face pass everywhere (before it: p = 4
  // FP32 16.4 -> 16.8 us, p = 6 FP64 +2 %).
  static constexpr int MIN_WAVES_EU = sizeof(T) == 4 ? 3 : 2;
  static constexpr bool EARLY_K = N <= 4;
};

// Stores of a LARGE launch (the stage's arrays exceed the last-level cache) do
// not displace what the neighbours still read; the cache policy of such a load.
constexpr int kNonTemporal = 2;
template <bool LARGE, typename V>
__device__ __forceinline__ void store(V* p, V v) {
  if constexpr (LARGE)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}

template <typename T>
struct FaceConst {  // wave-uniform constants of the pointwise physics
  Gas<T> gas;
  Base<T> base;
  T theta, k_wall, vwx, vwy;
};
template <typename T>
__device__ __forceinline__ FaceConst<T> face_const(const KernelPhysics& ph) {
  FaceConst<T> c;
  c.gas.gamma = (T)ph.gamma;
  c.gas.gm1 = (T)ph.gm1;
  c.gas.igm1 = (T)ph.igm1;
  c.gas.mu = (T)ph.mu;
  c.gas.k = (T)ph.k;
  c.base.rho = (T)ph.U_inf[0];
  c.base.mx = (T)ph.U_inf[1];
  c.base.my = (T)ph.U_inf[2];
  c.base.E = (T)ph.U_inf[3];
  c.base.p = (T)ph.p_inf;
  c.base.ux = (T)ph.u_inf;
  c.base.uy = (T)ph.v_inf;
  c.theta = (T)ph.theta;
  c.k_wall = (T)ph.k_wall;
  c.vwx = (T)ph.vw[0];
  c.vwy = (T)ph.vw[1];
  return c;
}

// The lane's face node: element slot, face, node along it, volume node.
template <int N, typename T, bool LARGE>
struct FaceLane {
  int e, fn, f, j, n;
  __device__ __forceinline__ explicit FaceLane(int lane) {
    using P = TraceOrder<N, T, LARGE>;
    e = lane / P::NF;
    fn = lane - e * P::NF;
    e = e < P::EPT ? e : P::EPT - 1;
    f = fn / P::Nfp;
    j = fn - f * P::Nfp;
    n = face_node<N>(f, j);
  }
};

// matrix-core row of (field c, element slot e)
template <int N, typename T, bool LARGE>
__device__ __forceinline__ int row_of(int c, int e) {
  using P = TraceOrder<N, T, LARGE>;
  return P::G == 1 ? P::ROWC * c + P::ROWE * e : (e >> 2) * 16 + P::ROWC * c + P::ROWE * (e & 3);
}

// Gradient of the staged states on the matrix cores: output lane (group g,
// slot l/16, node 16 tt + l%16) holds all four fields' x and y derivatives.
template <int N, typename T, bool LARGE>
__device__ __forceinline__ void tile_gradient(const T* sU, const T* sGeo, const T* sFrag, int lane,
                                              int nel, T (&gx)[TraceOrder<N, T, LARGE>::G][TraceOrder<N, T, LARGE>::NT][4],
                                              T (&gy)[TraceOrder<N, T, LARGE>::G][TraceOrder<N, T, LARGE>::NT][4]) {
  using P = TraceOrder<N, T, LARGE>;
  using O = Order<N, T>;
  typedef typename Vec4<T>::type V4;
  const int arow = lane & 15, acol = lane >> 4, re = lane >> 4, rn = lane & 15;
#pragma unroll
  for (int g = 0; g < P::G; ++g)
#pragma unroll
    for (int tt = 0; tt < P::NT; ++tt) {
      V4 aR = {T(0), T(0), T(0), T(0)}, aS = {T(0), T(0), T(0), T(0)};
#pragma unroll
      for (int s = 0; s < P::KS; ++s) {
        const T av = sU[(g * 16 + arow) * P::RS + 4 * s + acol];
        aR = mfma(av, sFrag[(tt * P::KS + s) * 64 + lane], aR);
        aS = mfma(av, sFrag[O::FD + (tt * P::KS + s) * 64 + lane], aS);
      }
      const int e = 4 * g + re;
      const bool ok = e < nel && 16 * tt + rn < P::Np;
      const T* m = sGeo + e * kGeoStride;
      const T rx = ok ? m[0] : T(0), ry = ok ? m[1] : T(0);
      const T sx = ok ? m[2] : T(0), sy = ok ? m[3] : T(0);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        gx[g][tt][c] = rx * aR[c] + sx * aS[c];
        gy[g][tt][c] = ry * aR[c] + sy * aS[c];
      }
    }
}

// The gradient at node n of element slot e, from the lane that holds it.
template <int N, typename T, bool LARGE>
__device__ __forceinline__ void fetch_gradient(const T (&gxk)[TraceOrder<N, T, LARGE>::G][TraceOrder<N, T, LARGE>::NT][4],
                                               const T (&gyk)[TraceOrder<N, T, LARGE>::G][TraceOrder<N, T, LARGE>::NT][4],
                                               int e, int n, T gx[4], T gy[4]) {
  using P = TraceOrder<N, T, LARGE>;
  const int src = 16 * (e & 3) + (n & 15);
#pragma unroll
  for (int g = 0; g < P::G; ++g)
#pragma unroll
    for (int tt = 0; tt < P::NT; ++tt) {
      const bool here = (P::G == 1 || (e >> 2) == g) && (P::NT == 1 || (n >> 4) == tt);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const T vx = lane_read(gxk[g][tt][c], src), vy = lane_read(gyk[g][tt][c], src);
        if (here) {
          gx[c] = vx;
          gy[c] = vy;
        }
      }
    }
}

// Zero the pad columns of `rows` rows of RS values.  The matrix-core products
// read them against zero operator entries, and 0 times a NaN or an infinity is
// not 0: a row is one element's, its pads must be no other's.  (Per tile: 0.994 to
// 1.008 of the steps' times with the pads cleared once a launch.)
template <int N, typename T>
__device__ __forceinline__ void zero_pads(T* rows0, int rows, int lane) {
  using P = TraceOrder<N, T>;
  if constexpr (P::PAD > 0)
    for (int i = lane; i < rows * P::PAD; i += 64) {
      const int r = i / P::PAD;
      rows0[r * P::RS + P::Np + (i - r * P::PAD)] = T(0);
    }
}

// The traces of the states staged in sU (synced): one lane per face node of
// the tile's nel elements.  Boundary faces carry the wall's or the far field's
// viscous flux, and the ghost's norm in the maximum.  skip: the slots (bits) whose
// traces another wave writes: their new states are not in sU, and what is formed
// of those rows stays in them (left out before the norm, 4 us of 990 slower at
// p = 4 FP32).
template <int N, typename T, bool PERT, bool LARGE>
__device__ __forceinline__ void write_traces(const FaceConst<T>& fc, const FaceLane<N, T, LARGE>& fl,
                                             const T* sU, const T* sGeo, T* sNorm, const T* sFrag,
                                             int lane, int conn, int nel, int64_t e0,
                                             typename Vec4<T>::type* __restrict__ tr, unsigned skip = 0) {
  using P = TraceOrder<N, T, LARGE>;
  T gxk[P::G][P::NT][4], gyk[P::G][P::NT][4];
  tile_gradient<N, T, LARGE>(sU, sGeo, sFrag, lane, nel, gxk, gyk);
  T gxp[4], gyp[4];
  fetch_gradient<N, T, LARGE>(gxk, gyk, fl.e, fl.n, gxp, gyp);
  const bool ok = lane < nel * P::NF;
  T vn[4] = {T(0), T(0), T(0), T(0)};
  T nrm = T(0);
  if (ok) {
    const int tag = conn & 3;
    const T* g = sGeo + fl.e * kGeoStride;
    const T nx = g[4 + 4 * fl.f], ny = g[5 + 4 * fl.f];
    T up[4], upf[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) up[c] = sU[row_of<N, T, LARGE>(c, fl.e) * P::RS + fl.n];
    full_state<T, PERT>(up, fc.base, upf);
    const VState<T> sp = vstate(fc.gas, upf);
    VState<T> so = sp;
    if (tag != 0) {
      T uo[4], uof[4];
      ghost_state<T, PERT>(tag, up, upf, nullptr, 0, fc.vwx, fc.vwy, fc.gas, fc.base, uo);
      full_state<T, PERT>(uo, fc.base, uof);
      so = vstate(fc.gas, uof);
    }
    // one evaluation for interior faces, a second for the ghosts
    const int sides = tag == 0 ? 1 : 2;
#pragma nounroll
    for (int side = 0; side < sides; ++side) {
      const T a1 = normal_diffusion_norm(fc.gas, side == 0 ? sp : so, nx, ny);
      nrm = a1 > nrm ? a1 : nrm;
    }
    if (tag == 1)
      viscous_normal_flux(gas_wall(fc.gas, fc.k_wall), so, gxp, gyp, nx, ny, vn);
    else
      viscous_normal_flux(fc.gas, sp, gxp, gyp, nx, ny, vn);
    sNorm[lane] = nrm;
  }
  wave_sync();
  if (ok && !((skip >> fl.e) & 1)) {
    T gmax = T(0);
#pragma unroll
    for (int jj = 0; jj < P::Nfp; ++jj) {
      const T v = sNorm[lane - fl.j + jj];
      gmax = v > gmax ? v : gmax;
    }
    store<LARGE>(tr + e0 * P::NF + lane, typename Vec4<T>::type{vn[1], vn[2], vn[3], gmax});
  }
}

// The stage for the tiles tile0, tile0 + stride, ... < tile_end of one mesh,
// run by one wavefront: traces tr_in of Uin in, and unless tr_out is null
// those of the new state out.  `lds_init` runs once, after the first tile's
// loads are issued (the workgroup's operator fragments, whose latency the
// loads then share).  CURVED: the elements of the curved set, whose outputs and
// traces other waves write, are left out of a tile's stores.
template <int N, typename T, bool PERT, bool LARGE, bool CURVED, typename Init>
__device__ __forceinline__ void trace_tiles(const DeviceTables& t, const KernelPhysics& ph,
                                            const double* __restrict__ Uin,
                                            double* __restrict__ Uout, double* __restrict__ K1,
                                            double a, double b, double dt,
                                            const typename Vec4<T>::type* __restrict__ tr_in,
                                            typename Vec4<T>::type* __restrict__ tr_out,
                                            const T* sFrag, T* area, int64_t tile0,
                                            int64_t tile_end, int64_t stride, Init lds_init) {
  using P = TraceOrder<N, T, LARGE>;
  using O = Order<N, T>;
  typedef typename Vec4<T>::type V4;
  constexpr int Np = P::Np, Nfp = P::Nfp, NF = P::NF, S = P::S, NT = P::NT, KS = P::KS, KF = P::KF,
                RS = P::RS, HRS = P::HRS, ROWC = P::ROWC, ROWE = P::ROWE, EPT = P::EPT, G = P::G,
                BE = P::BE, EB = P::EB, NQ = P::NQ, NG = P::NG;
  constexpr bool REREAD = PERT || P::OVER;  // K0 re-read in FP64 for the update
  constexpr int OFF_L = 2 * O::FD, OFF_LR = OFF_L + O::FL, OFF_LS = OFF_LR + O::FL;
  const int lane = threadIdx.x & 63;
  T* sU = area;
  T* sFr = area + P::U_SZ;
  T* sFs = sFr + G * 16 * RS;
  T* sH = area + P::H_OFF;
  T* sQr = sH + G * 16 * HRS;
  T* sQs = sQr + G * 16 * HRS;
  T* sNorm = sFr;
  T* sGeo = area + P::AREA;
  const FaceConst<T> fc = face_const<T>(ph);
  const FaceLane<N, T, LARGE> fl(lane);
  const int64_t K = t.K;
  const int arow = lane & 15, acol = lane >> 4, re = lane >> 4, rn = lane & 15;

  // state loads: value r = lane + 64 q of a run of BE element blocks
  int lds_u[NQ], field[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int r = lane + 64 * q, e = r / S, v = r - e * S, c = v / Np;
    lds_u[q] = row_of<N, T, LARGE>(c, e) * RS + (v - c * Np);
    field[q] = c;
  }
  // the free stream of field c, subtracted in the perturbation forms (selects
  // among values: an indexed read would put a copy of ph into scratch memory)
  const double ui0 = ph.U_inf[0], ui1 = ph.U_inf[1], ui2 = ph.U_inf[2], ui3 = ph.U_inf[3];
  auto uinf = [&](int c) -> double {
    const double lo = c == 0 ? ui0 : ui1, hi = c == 2 ? ui2 : ui3;
    return !PERT ? 0.0 : (c < 2 ? lo : hi);
  };
  double ru[EB][NQ], rg[NG];
  V4 rt = {};
  int rc = 0;
  // own states, geometry, connectivity and traces, through descriptors over
  // the tile's elements (past the last element a load reads 0, and such values
  // are never stored; a lane past its run reads a value it does not store)
  auto load_own = [&](int64_t tl) {
    const int64_t b0 = tl * EPT;
    const int64_t nb = K - b0 < EPT ? K - b0 : EPT;
    const __amdgpu_buffer_rsrc_t ud = records(Uin, b0, nb, S * 8);
#pragma unroll
    for (int eb = 0; eb < EB; ++eb)
#pragma unroll
      for (int q = 0; q < NQ; ++q) ru[eb][q] = buf_load_f64(ud, (eb * S + lane + 64 * q) * 8);
    const __amdgpu_buffer_rsrc_t gd = records(t.geo, b0, nb, kGeoStride * 8);
#pragma unroll
    for (int q = 0; q < NG; ++q) rg[q] = buf_load_f64(gd, (lane + 64 * q) * 8);
    rc = __builtin_amdgcn_raw_buffer_load_b32(records(t.conn, b0, nb, 3 * 4), lane * 4, 0, 0);
    const __amdgpu_buffer_rsrc_t td = records(tr_in, b0, nb, NF * (int)sizeof(V4));
    if constexpr (sizeof(T) == 4) {
      rt = __builtin_bit_cast(V4, __builtin_amdgcn_raw_buffer_load_b128(td, lane * 16, 0, 0));
    } else {
      typedef double D2 __attribute__((ext_vector_type(2)));
      const D2 lo = __builtin_bit_cast(D2, __builtin_amdgcn_raw_buffer_load_b128(td, lane * 32, 0, 0));
      const D2 hi = __builtin_bit_cast(D2, __builtin_amdgcn_raw_buffer_load_b128(td, lane * 32 + 16, 0, 0));
      rt = V4{lo.x, lo.y, hi.x, hi.y};
    }
  };
  load_own(tile0);
  lds_init();

  for (int64_t tile = tile0; tile < tile_end; tile += stride) {
    const int64_t e0 = tile * EPT;
    const int nel = (int)((K - e0) < EPT ? (K - e0) : EPT);
    wave_sync();
#pragma unroll
    for (int eb = 0; eb < EB; ++eb)
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const bool in = BE == 1 ? (lane + 64 * q < S && eb < nel) : (lane + 64 * q < nel * S);
        if (in) sU[lds_u[q] + ROWE * eb * RS] = (T)(ru[eb][q] - uinf(field[q]));
      }
#pragma unroll
    for (int q = 0; q < NG; ++q)
      if (lane + 64 * q < nel * kGeoStride) sGeo[lane + 64 * q] = (T)rg[q];
    // the last tile's face terms and norms lay on the flux rows (OVER: on the state
    // rows too)
    zero_pads<N, T>(P::OVER ? sU : sFr, P::OVER ? G * 48 : G * 32, lane);
    // the face node's other side: its state (4 strided values) and its trace;
    // a boundary face points at the element itself
    const bool okf = lane < nel * NF;
    // slots of the curved set
    unsigned skip = 0;
    if constexpr (CURVED) skip = (unsigned)__ballot(lane < nel && t.cslot[e0 + (lane < nel ? lane : 0)] >= 0);
    auto kept = [&](int e) { return !CURVED || !((skip >> e) & 1); };
    const int conn = __builtin_amdgcn_ds_bpermute((fl.e * 3 + fl.f) << 2, rc);
    const int tag = conn & 3;
    const V4 own = rt;
    double un[4];
    V4 nbt;
    {
      const int mf = tag == 0 ? (conn >> 2) & 3 : fl.f;
      const int mj = tag == 0 ? Nfp - 1 - fl.j : fl.j;
      const int64_t ne = okf ? (int64_t)(conn >> 4) : e0;
      const int mfo = okf ? mf : 0;
      const double* up = Uin + ne * S + face_node<N>(mfo, mj);
#pragma unroll
      for (int c = 0; c < 4; ++c) un[c] = up[c * Np];
      nbt = tr_in[ne * NF + mfo * Nfp + mj];
    }
    // (between elements of the set no traces are written: what those lanes read may
    // be anything, and stays in those elements' rows)
    wave_sync();

    // ---- gradient on the matrix cores, volume flux per node, contravariant
    auto volume_flux = [&](int e, int n, const T gx[4], const T gy[4]) {
      const T* g = sGeo + e * kGeoStride;
      const T rx = g[0], ry = g[1], sx = g[2], sy = g[3];
      T u[4], uf[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) u[c] = sU[row_of<N, T, LARGE>(c, e) * RS + n];
      full_state<T, PERT>(u, fc.base, uf);
      T fvx[4], fvy[4];
      const VState<T> st = vstate(fc.gas, uf);
      viscous_flux(fc.gas, st, gx, gy, fvx, fvy);
      const Prim<T> pr = prim_of<T, PERT>(uf, u, fc.base, fc.gas.gm1);
      T Fx[4], Fy[4];
      normal_flux<T, PERT>(uf, u, pr, fc.base, T(1), T(0), fc.vwx, Fx);
      normal_flux<T, PERT>(uf, u, pr, fc.base, T(0), T(1), fc.vwy, Fy);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const T fx = Fx[c] - fvx[c], fy = Fy[c] - fvy[c];
        sFr[row_of<N, T, LARGE>(c, e) * RS + n] = rx * fx + ry * fy;
        sFs[row_of<N, T, LARGE>(c, e) * RS + n] = sx * fx + sy * fy;
      }
    };
    {
      T gxk[G][NT][4], gyk[G][NT][4];
      tile_gradient<N, T, LARGE>(sU, sGeo, sFrag, lane, nel, gxk, gyk);
      if constexpr (P::PACK) {
        const int e = lane / Np, n = lane - e * Np;
        T gx[4], gy[4];
        fetch_gradient<N, T, LARGE>(gxk, gyk, e < EPT ? e : EPT - 1, n, gx, gy);
        if (e < nel) volume_flux(e, n, gx, gy);
      } else {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int tt = 0; tt < NT; ++tt)
            if (4 * g + re < nel && 16 * tt + rn < Np)
              volume_flux(4 * g + re, 16 * tt + rn, gxk[g][tt], gyk[g][tt]);
      }
    }
    wave_sync();

    // ---- K1 / K0 of the tile's outputs (output i: field i at the lane's node of
    // the matrix-core layout, or value lane + 64 i of the run)
    constexpr int NO = P::FLAT ? NQ : 4;
    double rk[NO], r0[NO];
    auto out_off = [&](int i) { return P::FLAT ? lane + 64 * i : re * S + i * Np + (rn < Np ? rn : Np - 1); };
    auto load_k = [&] {
      const __amdgpu_buffer_rsrc_t rk_d = records(a != 0.0 ? K1 : Uin, e0, nel, S * 8);
      const __amdgpu_buffer_rsrc_t r0_d = records(Uin, e0, nel, S * 8);
#pragma unroll
      for (int i = 0; i < NO; ++i) {
        rk[i] = __builtin_bit_cast(
            double, __builtin_amdgcn_raw_buffer_load_b64(rk_d, out_off(i) * 8, 0, LARGE ? kNonTemporal : 0));
        r0[i] = REREAD ? buf_load_f64(r0_d, out_off(i) * 8) : 0.0;
      }
    };
    if constexpr (P::EARLY_K) load_k();

    // ---- the face node's own state and flux, then the divergence on the
    // matrix cores: after it the flux rows are free for the face terms
    T up[4] = {T(0), T(0), T(0), T(0)}, fr[4] = {T(0), T(0), T(0), T(0)}, fs[4] = {T(0), T(0), T(0), T(0)};
    if (okf) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int i = row_of<N, T, LARGE>(c, fl.e) * RS + fl.n;
        up[c] = sU[i];
        fr[c] = sFr[i];
        fs[c] = sFs[i];
      }
    }
    V4 aD[G][NT];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int tt = 0; tt < NT; ++tt) {
        aD[g][tt] = V4{T(0), T(0), T(0), T(0)};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          const int ao = (g * 16 + arow) * RS + 4 * s + acol, fo = (tt * KS + s) * 64 + lane;
          aD[g][tt] = mfma(sFr[ao], sFrag[fo], aD[g][tt]);
          aD[g][tt] = mfma(sFs[ao], sFrag[O::FD + fo], aD[g][tt]);
        }
      }
    wave_sync();

    // ---- face nodes, one lane each
    if (okf) {
      const T* g = sGeo + fl.e * kGeoStride;
      const T nx = g[4 + 4 * fl.f], ny = g[5 + 4 * fl.f], fsc = g[6 + 4 * fl.f];
      T uo[4], upf[4], uof[4], unb[4];
      full_state<T, PERT>(up, fc.base, upf);
#pragma unroll
      for (int c = 0; c < 4; ++c) unb[c] = (T)(PERT ? un[c] - ph.U_inf[c] : un[c]);
      ghost_state<T, PERT>(tag, up, upf, unb, 1, fc.vwx, fc.vwy, fc.gas, fc.base, uo);
      full_state<T, PERT>(uo, fc.base, uof);
      // mean viscous normal flux (the other side's normal is -n); one side's
      // on a boundary face
      const T vn[4] = {T(0), tag == 0 ? T(0.5) * (own[0] - nbt[0]) : own[0],
                       tag == 0 ? T(0.5) * (own[1] - nbt[1]) : own[1],
                       tag == 0 ? T(0.5) * (own[2] - nbt[2]) : own[2]};
      const T gbar = nbt[3] > own[3] ? nbt[3] : own[3];
      const T sigma = g[7 + 4 * fl.f] * gbar;
      const T vwn = fc.vwx * nx + fc.vwy * ny;
      const Prim<T> pp = prim_of<T, PERT>(upf, up, fc.base, fc.gas.gm1);
      T Fc[4];
      if (tag == 1) {
        // pressure through the moving wall (minus the free-stream flux in the
        // perturbation form)
        if (!PERT) {
          Fc[0] = T(0);
          Fc[1] = pp.p * nx;
          Fc[2] = pp.p * ny;
          Fc[3] = pp.p * vwn;
        } else {
          const T q0n = fc.base.ux * nx + fc.base.uy * ny - vwn;
          Fc[0] = -fc.base.rho * q0n;
          Fc[1] = pp.jp * nx - fc.base.mx * q0n;
          Fc[2] = pp.jp * ny - fc.base.my * q0n;
          Fc[3] = pp.jp * vwn - (fc.base.E + fc.base.p) * q0n;
        }
      } else {
        const Prim<T> po = prim_of<T, PERT>(uof, uo, fc.base, fc.gas.gm1);
        T FL[4], FR[4];
        normal_flux<T, PERT>(upf, up, pp, fc.base, nx, ny, vwn, FL);
        normal_flux<T, PERT>(uof, uo, po, fc.base, nx, ny, vwn, FR);
        roe_flux(pp, po, FL, FR, nx, ny, vwn, fc.gas.gm1, Fc);
      }
      // Fscale * own total normal flux from the contravariant flux:
      // face 0: -Fs, face 1: Fr + Fs, face 2: -Fr
      const T cfr = fl.f == 0 ? T(0) : (fl.f == 1 ? T(1) : T(-1));
      const T cfs = fl.f == 2 ? T(0) : (fl.f == 1 ? T(1) : T(-1));
      T w[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const T ownf = cfr * fr[c] + cfs * fs[c];
        w[c] = up[c] - uo[c];
        sH[row_of<N, T, LARGE>(c, fl.e) * HRS + fl.fn] = ownf - fsc * (Fc[c] - vn[c] + sigma * w[c]);
      }
      T qx[4], qy[4];
      const VState<T> st = vstate(fc.gas, tag == 1 ? uof : upf);
      viscous_transpose(tag == 1 ? gas_wall(fc.gas, fc.k_wall) : fc.gas, st, nx, ny, w, qx, qy);
      const T ce = fc.theta * (tag == 0 ? T(0.5) : T(1)) * fsc;
      const T rx = g[0], ry = g[1], sx = g[2], sy = g[3];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        sQr[row_of<N, T, LARGE>(c, fl.e) * HRS + fl.fn] = ce * (rx * qx[c] + ry * qy[c]);
        sQs[row_of<N, T, LARGE>(c, fl.e) * HRS + fl.fn] = ce * (sx * qx[c] + sy * qy[c]);
      }
    }
    for (int i = lane; i < G * 48 * (HRS - NF); i += 64) {
      const int row = i / (HRS - NF);
      sH[row * HRS + NF + (i - row * (HRS - NF))] = T(0);
    }
    wave_sync();
    if constexpr (!P::EARLY_K) load_k();
    load_own(tile + stride);

    // ---- lifts on the matrix cores, then the RK stage in FP64
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int tt = 0; tt < NT; ++tt) {
        V4 aL = {T(0), T(0), T(0), T(0)};
#pragma unroll
        for (int s = 0; s < KF; ++s) {
          const int fi = (tt * KF + s) * 64 + lane, ao = (g * 16 + arow) * HRS + 4 * s + acol;
          aL = mfma(sH[ao], sFrag[OFF_L + fi], aL);
          aL = mfma(sQr[ao], sFrag[OFF_LR + fi], aL);
          aL = mfma(sQs[ao], sFrag[OFF_LS + fi], aL);
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) aD[g][tt][c] = aL[c] - aD[g][tt][c];
      }
    if constexpr (P::FLAT) {
      wave_sync();
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
          if (16 * tt + rn < Np && 4 * g + re < EPT) {
#pragma unroll
            for (int c = 0; c < 4; ++c) sH[row_of<N, T, LARGE>(c, 4 * g + re) * RS + 16 * tt + rn] = aD[g][tt][c];
          }
      wave_sync();
    }
    double unew[NO];
#pragma unroll
    for (int i = 0; i < NO; ++i) {
      const int at = P::FLAT ? lds_u[P::FLAT ? i : 0] : row_of<N, T, LARGE>(i, re) * RS + rn;
      const bool in = (P::FLAT ? lane + 64 * i < nel * S : (re < nel && rn < Np));
      if (in && kept(P::FLAT ? (lane + 64 * i) / S : re)) {
        const double R = (double)(P::FLAT ? sH[at] : aD[0][0][P::FLAT ? 0 : i]);
        const int64_t idx = e0 * S + out_off(i);
        const double k = (a != 0.0) ? a * rk[i] + dt * R : dt * R;
        store<LARGE>(K1 + idx, k);
        const double u0 = REREAD ? r0[i] : (double)sU[at];
        unew[i] = u0 + b * k;
        store<LARGE>(Uout + idx, unew[i]);
      }
    }
    if (tr_out != nullptr) {
      // ---- the new state's traces for the next stage
      wave_sync();
#pragma unroll
      for (int i = 0; i < NO; ++i) {
        const int at = P::FLAT ? lds_u[P::FLAT ? i : 0] : row_of<N, T, LARGE>(i, re) * RS + rn;
        const bool in = P::FLAT ? lane + 64 * i < nel * S : (re < nel && rn < Np);
        if (in && kept(P::FLAT ? (lane + 64 * i) / S : re)) sU[at] = (T)(unew[i] - uinf(P::FLAT ? field[P::FLAT ? i : 0] : i));
      }
      if constexpr (P::OVER) zero_pads<N, T>(sU, G * 16, lane);
      wave_sync();
      write_traces<N, T, PERT, LARGE>(fc, fl, sU, sGeo, sNorm, sFrag, lane, conn, nel, e0, tr_out, skip);
    }
  }
}

// Copy COUNT operator fragment values into LDS and zero the pad columns of the
// workgroup's state and flux rows.
template <int N, typename T, int W, int COUNT, bool LARGE, int WS>
__device__ __forceinline__ void trace_lds_init(const T* __restrict__ frag, T* sFrag, T* sWave) {
  using P = TraceOrder<N, T, LARGE>;
  copy_to_lds<COUNT, W>(frag, sFrag);
  zero_pads<N, T>(sWave + (threadIdx.x >> 6) * WS, P::G * 48, threadIdx.x & 63);
  __syncthreads();
}

template <typename T>
__device__ __forceinline__ const T* frag_table(const DeviceTables& t);
template <>
__device__ __forceinline__ const double* frag_table<double>(const DeviceTables& t) {
  return t.frag;
}
template <>
__device__ __forceinline__ const float* frag_table<float>(const DeviceTables& t) {
  return t.frag32;
}

// One wave's tile of the traces of a given state (the first stage of a call):
// states, geometry and connectivity into LDS, then the traces.
template <int N, typename T, bool PERT, bool LARGE>
__device__ __forceinline__ void trace_tile(const DeviceTables& t, const KernelPhysics& ph,
                                           const double* __restrict__ U,
                                           typename Vec4<T>::type* __restrict__ tr, const T* sFrag,
                                           T* area, int64_t tile) {
  using P = TraceOrder<N, T, LARGE>;
  const int lane = threadIdx.x & 63;
  T* sU = area;
  T* sGeo = area + P::AREA;
  const FaceConst<T> fc = face_const<T>(ph);
  const FaceLane<N, T, LARGE> fl(lane);
  const int64_t e0 = tile * P::EPT;
  const int nel = (int)((t.K - e0) < P::EPT ? (t.K - e0) : P::EPT);
  const __amdgpu_buffer_rsrc_t ud = records(U, e0, nel, P::S * 8);
  const __amdgpu_buffer_rsrc_t gd = records(t.geo, e0, nel, kGeoStride * 8);
  constexpr int NQ = (P::EPT * P::S + 63) / 64;
  double ru[NQ], rg[P::NG];
#pragma unroll
  for (int q = 0; q < NQ; ++q) ru[q] = buf_load_f64(ud, (lane + 64 * q) * 8);
#pragma unroll
  for (int q = 0; q < P::NG; ++q) rg[q] = buf_load_f64(gd, (lane + 64 * q) * 8);
  const int conn =
      __builtin_amdgcn_raw_buffer_load_b32(records(t.conn, e0, nel, 3 * 4), (fl.e * 3 + fl.f) * 4, 0, 0);
  const double ui0 = ph.U_inf[0], ui1 = ph.U_inf[1], ui2 = ph.U_inf[2], ui3 = ph.U_inf[3];
  wave_sync();
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int r = lane + 64 * q, e = r / P::S, v = r - e * P::S, c = v / P::Np;
    const double lo = c == 0 ? ui0 : ui1, hi = c == 2 ? ui2 : ui3;
    if (r < nel * P::S)
      sU[row_of<N, T, LARGE>(c, e) * P::RS + (v - c * P::Np)] = (T)(ru[q] - (!PERT ? 0.0 : (c < 2 ? lo : hi)));
  }
#pragma unroll
  for (int q = 0; q < P::NG; ++q)
    if (lane + 64 * q < nel * kGeoStride) sGeo[lane + 64 * q] = (T)rg[q];
  wave_sync();
  write_traces<N, T, PERT, LARGE>(fc, fl, sU, sGeo, sU + P::U_SZ, sFrag, lane, conn, nel, e0, tr);
}

// The viscous normal flux and the norm at node (f, j) of element k, whose state
// is u ([4][Np]), on the lane itself, in the operations of write_traces: the
// gradient is the matrix cores' chain of fused multiply-adds over the element's
// nodes.  WALL: with the wall's ghost; else the element's own side alone.
template <int N, typename T, bool PERT, bool WALL>
__device__ __forceinline__ T node_trace(const DeviceTables& t, const KernelPhysics& ph, const FaceConst<T>& fc,
                                        const double* u, int64_t k, int f, int j, T vn[4]) {
  using P = TraceOrder<N, T>;
  using O = Order<N, T>;
  const T* frag = frag_table<T>(t);
  const int n = face_node<N>(f, j);
  T ur[4] = {T(0), T(0), T(0), T(0)}, us[4] = {T(0), T(0), T(0), T(0)};
  const int at = ((n >> 4) * P::KS) * 64 + (n & 15);
#pragma unroll 8
  for (int m = 0; m < P::Np; ++m) {
    const int fi = at + (m >> 2) * 64 + (m & 3) * 16;
    const T dr = frag[fi], ds = frag[O::FD + fi];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const T v = (T)(u[c * P::Np + m] - (PERT ? ph.U_inf[c] : 0.0));
      ur[c] += dr * v;
      us[c] += ds * v;
    }
  }
  const double* g = t.geo + k * kGeoStride;
  const T rx = (T)g[0], ry = (T)g[1], sx = (T)g[2], sy = (T)g[3];
  const T nx = (T)g[4 + 4 * f], ny = (T)g[5 + 4 * f];
  T gx[4], gy[4], up[4], upf[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    gx[c] = rx * ur[c] + sx * us[c];
    gy[c] = ry * ur[c] + sy * us[c];
    up[c] = (T)(u[c * P::Np + n] - (PERT ? ph.U_inf[c] : 0.0));
  }
  full_state<T, PERT>(up, fc.base, upf);
  const VState<T> sp = vstate(fc.gas, upf);
  VState<T> so = sp;
  if constexpr (WALL) {
    T uo[4], uof[4];
    ghost_state<T, PERT>(1, up, upf, nullptr, 0, fc.vwx, fc.vwy, fc.gas, fc.base, uo);
    full_state<T, PERT>(uo, fc.base, uof);
    so = vstate(fc.gas, uof);
  }
  T nrm = T(0);
#pragma nounroll
  for (int side = 0; side < (WALL ? 2 : 1); ++side) {
    const T a1 = normal_diffusion_norm(fc.gas, side == 0 ? sp : so, nx, ny);
    nrm = a1 > nrm ? a1 : nrm;
  }
  if constexpr (WALL)
    viscous_normal_flux(gas_wall(fc.gas, fc.k_wall), so, gx, gy, nx, ny, vn);
  else
    viscous_normal_flux(fc.gas, sp, gx, gy, nx, ny, vn);
  return nrm;
}

// Node (f, j)'s trace into place, with the largest of its face's norms, which lie
// in `norms` by lane.
template <int N, typename T>
__device__ __forceinline__ void store_node_trace(typename Vec4<T>::type* __restrict__ tr, int64_t k, int f, int j,
                                                 const T vn[4], const T* norms, int lane) {
  using P = TraceOrder<N, T>;
  T gmax = T(0);
#pragma unroll
  for (int jj = 0; jj < P::Nfp; ++jj) {
    const T v = norms[lane - j + jj];
    gmax = v > gmax ? v : gmax;
  }
  tr[k * P::NF + f * P::Nfp + j] = typename Vec4<T>::type{vn[1], vn[2], vn[3], gmax};
}

// The traces of the wall faces alone, for a wall velocity other than the one
// they were written with: one lane per face node of the faces blk * F ..., F =
// 64 / (p + 1), of the wall face list.  norms: 64 values of LDS.
template <int N, typename T, bool PERT>
__device__ __forceinline__ void wall_traces(const DeviceTables& t, const KernelPhysics& ph,
                                            const double* __restrict__ U,
                                            typename Vec4<T>::type* __restrict__ tr, int blk, T* norms) {
  using P = TraceOrder<N, T>;
  const int lane = threadIdx.x & 63;
  const int wf = blk * (64 / P::Nfp) + lane / P::Nfp, j = lane % P::Nfp;
  const bool ok = lane < 64 / P::Nfp * P::Nfp && wf < t.nwall;
  const FaceConst<T> fc = face_const<T>(ph);
  T vn[4] = {T(0), T(0), T(0), T(0)};
  int64_t k = 0;
  int f = 0;
  if (ok) {
    const int kf = t.wall[wf];
    k = kf / 3;
    f = kf % 3;
    norms[lane] = node_trace<N, T, PERT, true>(t, ph, fc, U + k * P::S, k, f, j, vn);
  }
  wave_sync();
  if (ok) store_node_trace<N, T>(tr, k, f, j, vn, norms, lane);
}

// The traces of one element of the curved set towards its straight neighbours,
// from its state u (in LDS, synced).  The set holds the isoparametric elements'
// face neighbours too, so those neighbours face an affine element: its traces are
// those of any straight one.  Nobody reads the set's other traces.  norms: 64
// values of LDS.
template <int N, typename T, bool PERT>
__device__ __forceinline__ void element_traces(const DeviceTables& t, const KernelPhysics& ph, const double* u,
                                               int64_t k, typename Vec4<T>::type* __restrict__ tr, T* norms) {
  using P = TraceOrder<N, T>;
  const int lane = threadIdx.x & 63;
  const int f = lane / P::Nfp, j = lane % P::Nfp;
  bool ok = false;
  if (lane < P::NF) {
    const int conn = t.conn[k * 3 + f];
    ok = (conn & 3) == 0 && t.cslot[conn >> 4] < 0;
  }
  const FaceConst<T> fc = face_const<T>(ph);
  T vn[4] = {T(0), T(0), T(0), T(0)};
  if (ok) norms[lane] = node_trace<N, T, PERT, false>(t, ph, fc, u, k, f, j, vn);
  wave_sync();
  if (ok) store_node_trace<N, T>(tr, k, f, j, vn, norms, lane);
}

namespace {
// The arrays a stage touches (U_in, U_out, K1, traces in and out, geometry) against
// the 256 MB last-level cache.  Where they fit, the next stage finds them
// there; beyond it, outputs and K1 stored and read past the caches' normal
// allocation (and in whole lines) leave the L2 to the neighbours' states:
// cylinder327k p = 4 FP32 (1 GB) 228 -> 204 us a stage, cylinder20k (63 MB) 16.4
// -> 17.7 us.
constexpr int64_t kLastLevelCache = int64_t(256) << 20;
constexpr int64_t stage_bytes(int N, int size, int64_t K) {
  return K * (3 * 8 * 4 * ((N + 1) * (N + 2) / 2) + 2 * 4 * size * 3 * (N + 1) + 8 * kGeoStride);
}
}  // namespace

}  // namespace dgmi
