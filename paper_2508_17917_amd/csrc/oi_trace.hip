// The over-integrated stage (FP64, degree-3p quadrature) from face traces, in
// multi-step calls.  As on the nodal stage, every element leaves for the next
// one what its neighbours need of it: per face point its own value (4), its
// viscous normal flux (3; the first is zero) and the face's largest norm -- 8
// doubles, [K][3q][8].  A neighbour's point is the mirrored one, its normal
// the own one negated, and both sides interpolate with the same weights in
// the same order, so the bits are those of the stage that evaluates both
// sides (kernels.hip).
//
// That stage ran one wave per SIMD (the neighbours' blocks in LDS, both sides'
// gradients on the vector unit, 50 KB of operator fragments per tile from the
// L2).  Here a wave needs half the LDS, so two run per SIMD; up to p = 4 the
// fragments sit in LDS too (at p = 4 eight waves of 12 KB share them and fill a
// CU's 160 KB); at p >= 5 (88 and 151 KB) they are read from the L2 as before.
//
// us a stage on 20,480 elements, that stage -> this: p = 1 21.5 -> 15.4, p = 2
// 25.7 -> 21.6, p = 3 45.6 -> 27.1, p = 4 89.4 -> 54.2, p = 5 186.6 -> 113.2, p = 6
// 404 -> 346.  Bound by the FP64 units, which the matrix and the vector
// instructions share: at p = 4 78 matrix instructions of 64 cycles (a quarter of
// their rows idle: three of four element slots) and 1,440 vector instructions of
// 4 and more a tile, 6.7 tiles a SIMD.
#include <hip/hip_runtime.h>

#include "trace_device.h"

namespace dgmi {

template <int N>
struct OITrace {
  using P = OIOrder<N>;
  static constexpr bool LDS_FRAG = N <= 4;
  // face terms over the flux chunk; at p = 6 over the state rows too (K0
  // re-read), for two workgroups on a CU
  static constexpr bool OVER = N >= 6;
  // the traces are loaded before the element points where the registers hold
  // them through those
  static constexpr bool LATE = N >= 5;
  static constexpr int H_OFF = OVER ? 0 : P::U_SZ;
  static constexpr int AREA =
      P::U_SZ + P::F_SZ > H_OFF + P::H_SZ ? P::U_SZ + P::F_SZ : H_OFF + P::H_SZ;
  static constexpr int WAVE_SZ = (AREA + P::EPT * kGeoStride + 3) / 4 * 4;
  static constexpr int NQ = (P::EPT * P::S + 63) / 64;
  // one point beyond whole chunks (p = 4: 49) and a free element slot: no chunk of
  // its own
  static constexpr bool TAIL = P::Nq % 16 == 1 && P::EPT < 4 && 12 * P::EPT <= 64;
  static constexpr int CHUNKS = TAIL ? P::NQT - 1 : P::NQT;
  static constexpr int TAB = LDS_FRAG ? P::TOTAL : P::LDS_TAB;  // shared LDS (doubles)
  static constexpr int OFF_TAB = LDS_FRAG ? P::OFF_DRSF : 0;    // face-point tables in it
  static constexpr int FIRST = LDS_FRAG ? 0 : P::OFF_DRSF;      // its first value in the packed array
};

typedef double D2 __attribute__((ext_vector_type(2)));

// The lane's face point: element slot, point, face, point along it.
template <int N>
struct PointLane {
  int e, fg, f, gp;
  __device__ __forceinline__ explicit PointLane(int lane) {
    using P = OIOrder<N>;
    e = lane / P::NG;
    fg = lane - e * P::NG;
    e = e < P::EPT ? e : P::EPT - 1;
    f = fg / P::q;
    gp = fg - f * P::q;
  }
};

// The traces of the states staged in sU (synced).
template <int N>
__device__ __forceinline__ void write_point_traces(const FaceConst<double>& fc, const PointLane<N>& pl,
                                                   const double* sU, const double* sGeo, double* sNorm,
                                                   const double* sTab, int lane, int conn, int nel,
                                                   int64_t e0, D2* __restrict__ tr) {
  using P = OIOrder<N>;
  using O = Order<N, double>;
  constexpr int Np = P::Np, Nfp = P::Nfp, RS = P::RS, ROWC = O::ROWC, ROWE = O::ROWE;
  const double* sDRS = sTab;
  const double* sIf1 = sTab + 2 * P::NG * Np;
  const bool ok = lane < nel * P::NG;
  double up[4] = {0.0, 0.0, 0.0, 0.0}, vn[4] = {0.0, 0.0, 0.0, 0.0};
  if (ok) {
    const int tag = conn & 3;
    const double* g = sGeo + pl.e * kGeoStride;
    const double nx = g[4 + 4 * pl.f], ny = g[5 + 4 * pl.f];
    double ur[4] = {0.0, 0.0, 0.0, 0.0}, us[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 5
    for (int j = 0; j < Np; ++j) {
      const double dr = sDRS[2 * (pl.fg * Np + j)], ds = sDRS[2 * (pl.fg * Np + j) + 1];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const double v = sU[(ROWC * c + ROWE * pl.e) * RS + j];
        ur[c] += dr * v;
        us[c] += ds * v;
      }
    }
#pragma unroll
    for (int i = 0; i < Nfp; ++i) {
      const double w = sIf1[pl.gp * Nfp + i];
      const int n = face_node<N>(pl.f, i);
#pragma unroll
      for (int c = 0; c < 4; ++c) up[c] += w * sU[(ROWC * c + ROWE * pl.e) * RS + n];
    }
    double gx[4], gy[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      gx[c] = g[0] * ur[c] + g[2] * us[c];
      gy[c] = g[1] * ur[c] + g[3] * us[c];
    }
    const VState<double> sp = vstate(fc.gas, up);
    VState<double> so = sp;
    if (tag != 0) {
      double uo[4];
      ghost_state<double, false>(tag, up, up, nullptr, 1, fc.vwx, fc.vwy, fc.gas, fc.base, uo);
      so = vstate(fc.gas, uo);
    }
    const int sides = tag == 0 ? 1 : 2;
    double nrm = 0.0;
#pragma nounroll
    for (int side = 0; side < sides; ++side) {
      const double a1 = normal_diffusion_norm(fc.gas, side == 0 ? sp : so, nx, ny);
      nrm = a1 > nrm ? a1 : nrm;
    }
    sNorm[lane] = nrm;
    if (tag == 1)
      viscous_normal_flux(gas_wall(fc.gas, fc.k_wall), so, gx, gy, nx, ny, vn);
    else
      viscous_normal_flux(fc.gas, sp, gx, gy, nx, ny, vn);
  }
  wave_sync();
  if (ok) {
    double gmax = 0.0;
#pragma unroll
    for (int jj = 0; jj < P::q; ++jj) {
      const double v = sNorm[lane - pl.gp + jj];
      gmax = v > gmax ? v : gmax;
    }
    D2* o = tr + (e0 * P::NG + lane) * 4;
    o[0] = D2{up[0], up[1]};
    o[1] = D2{up[2], up[3]};
    o[2] = D2{vn[1], vn[2]};
    o[3] = D2{vn[3], gmax};
  }
}

template <int N>
__device__ __forceinline__ void zero_state_pads(double* sU, int lane) {
  using P = OIOrder<N>;
  constexpr int PAD = P::RS - P::Np;
  for (int i = lane; i < 16 * PAD; i += 64) sU[i / PAD * P::RS + P::Np + i % PAD] = 0.0;
}

// The state's loads of a tile: value lane + 64 q of its run of element blocks.
template <int N>
struct StateRun {
  int at[OITrace<N>::NQ];
  __device__ __forceinline__ explicit StateRun(int lane) {
    using P = OIOrder<N>;
    using O = Order<N, double>;
#pragma unroll
    for (int q = 0; q < OITrace<N>::NQ; ++q) {
      const int r = lane + 64 * q, e = r / P::S, v = r - e * P::S, c = v / P::Np;
      at[q] = (O::ROWC * c + O::ROWE * e) * P::RS + (v - c * P::Np);
    }
  }
};

template <int N>
__device__ __forceinline__ void oi_trace_tiles(const DeviceTables& t, const KernelPhysics& ph,
                                               const double* __restrict__ Uin, double* __restrict__ Uout,
                                               double* __restrict__ K1, double a, double b, double dt,
                                               const D2* __restrict__ tr_in, D2* __restrict__ tr_out,
                                               const double* sTabs, double* area, int64_t tile0,
                                               int64_t tile_end, int64_t stride) {
  using P = OIOrder<N>;
  using Q = OITrace<N>;
  using O = Order<N, double>;
  typedef Vec4<double>::type V4;
  constexpr int Np = P::Np, S = P::S, NT = P::NT, KS = P::KS, RS = P::RS, q = P::q, Nq = P::Nq, NG = P::NG,
                NQT = P::NQT, KQ = P::KQ, KG = P::KG, EPT = P::EPT, FRS = P::FRS, GRS = P::GRS,
                ROWC = O::ROWC, ROWE = O::ROWE, NQ = Q::NQ;
  const int lane = threadIdx.x & 63;
  const double* G = Q::LDS_FRAG ? sTabs : t.oi;
  const double* sTab = sTabs + Q::OFF_TAB;
  double* sU = area;
  double* sF = area + P::U_SZ;  // flux chunk: F_r rows | F_s rows; later the norms
  double* sH = area + Q::H_OFF;
  double* sQr = sH + 16 * GRS;
  double* sQs = sH + 32 * GRS;
  double* sGeo = area + Q::AREA;
  const FaceConst<double> fc = face_const<double>(ph);
  const PointLane<N> pl(lane);
  const StateRun<N> run(lane);
  const int64_t K = t.K;
  const int arow = lane & 15, acol = lane >> 4, re = lane >> 4, rn = lane & 15;

  double ru[NQ], rg = 0.0;
  int rc = 0;
  auto load_own = [&](int64_t tl) {
    const int64_t b0 = tl * EPT;
    const int64_t nb = K - b0 < EPT ? K - b0 : EPT;
    const __amdgpu_buffer_rsrc_t ud = records(Uin, b0, nb, S * 8);
#pragma unroll
    for (int i = 0; i < NQ; ++i) ru[i] = buf_load_f64(ud, (lane + 64 * i) * 8);
    rg = buf_load_f64(records(t.geo, b0, nb, kGeoStride * 8), lane * 8);
    rc = __builtin_amdgcn_raw_buffer_load_b32(records(t.conn, b0, nb, 3 * 4), lane * 4, 0, 0);
  };
  load_own(tile0);

  for (int64_t tile = tile0; tile < tile_end; tile += stride) {
    const int64_t e0 = tile * EPT;
    const int nel = (int)((K - e0) < EPT ? (K - e0) : EPT);
    wave_sync();
#pragma unroll
    for (int i = 0; i < NQ; ++i)
      if (lane + 64 * i < nel * S) sU[run.at[i]] = ru[i];
    if (lane < nel * kGeoStride) sGeo[lane] = rg;
    if constexpr (Q::OVER) zero_state_pads<N>(sU, lane);
    // own and neighbour traces of the lane's face point, for the face pass
    const bool ok = lane < nel * NG;
    const int conn = __builtin_amdgcn_ds_bpermute((pl.e * 3 + pl.f) << 2, rc);
    const int tag = conn & 3;
    D2 own[4], nbt[4];
    auto load_traces = [&] {
      const __amdgpu_buffer_rsrc_t td = records(tr_in, e0, nel, NG * 64);
      const int mf = tag == 0 ? (conn >> 2) & 3 : pl.f, mj = tag == 0 ? q - 1 - pl.gp : pl.gp;
      const D2* nb = tr_in + ((ok ? (int64_t)(conn >> 4) : e0) * NG + (ok ? mf : 0) * q + mj) * 4;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        own[i] = __builtin_bit_cast(D2, __builtin_amdgcn_raw_buffer_load_b128(td, lane * 64 + 16 * i, 0, 0));
        nbt[i] = nb[i];
      }
    };
    if constexpr (!Q::LATE) load_traces();
    wave_sync();

    // ---- element points, chunk by chunk; the divergence accumulates in acc.
    // TAIL: the last point's 12 values per element (U, d_r U, d_s U) are dot
    // products, one a lane, in the order of the matrix cores' chain; the free
    // slot's lanes form its flux with the first chunk's, and its share of the
    // divergence follows the other points' on the vector unit.  p = 4, 20,480
    // elements: 57.3 us a stage with a chunk for the one point, 54.2 without.
    if constexpr (Q::TAIL) {
      const int op = lane / (4 * EPT), r = lane - op * (4 * EPT), c = r / EPT, e = r - c * EPT;
      if (op < 3) {
        const double* fr = G + (op == 0 ? P::OFF_IQ : (op == 1 ? P::OFF_DRQ : P::OFF_DSQ)) + (NQT - 1) * KS * 64;
        const double* u = sU + (ROWC * c + ROWE * e) * RS;
        double v = 0.0;
#pragma unroll
        for (int k = 0; k < Np; ++k) v = __builtin_fma(u[k], fr[(k >> 2) * 64 + (k & 3) * 16], v);
        sF[lane] = v;
      }
      wave_sync();
    }
    double tFr[4] = {0.0, 0.0, 0.0, 0.0}, tFs[4] = {0.0, 0.0, 0.0, 0.0};
    V4 acc[NT];
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) acc[tt] = V4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int tq = 0; tq < Q::CHUNKS; ++tq) {
      V4 aU = {0.0, 0.0, 0.0, 0.0}, aR = aU, aS = aU;
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const double av = sU[arow * RS + 4 * s + acol];
        const int fo = (tq * KS + s) * 64 + lane;
        aU = mfma(av, G[P::OFF_IQ + fo], aU);
        aR = mfma(av, G[P::OFF_DRQ + fo], aR);
        aS = mfma(av, G[P::OFF_DSQ + fo], aS);
      }
      double Fr[4] = {0.0, 0.0, 0.0, 0.0}, Fs[4] = {0.0, 0.0, 0.0, 0.0};
      const bool tail = Q::TAIL && tq == 0 && re == EPT && rn < nel;
      if (tail) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          aU[c] = sF[c * EPT + rn];
          aR[c] = sF[(4 + c) * EPT + rn];
          aS[c] = sF[(8 + c) * EPT + rn];
        }
      }
      if (tail || (re < nel && 16 * tq + rn < Nq)) {
        const double* g = sGeo + (tail ? rn : re) * kGeoStride;
        const double rx = g[0], ry = g[1], sx = g[2], sy = g[3];
        double u[4], gx[4], gy[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          u[c] = aU[c];
          gx[c] = rx * aR[c] + sx * aS[c];
          gy[c] = ry * aR[c] + sy * aS[c];
        }
        double fvx[4], fvy[4], Fx[4], Fy[4];
        viscous_flux(fc.gas, vstate(fc.gas, u), gx, gy, fvx, fvy);
        const Prim<double> pr = prim_plain(u, fc.gas.gm1);
        normal_flux<double, false>(u, u, pr, fc.base, 1.0, 0.0, fc.vwx, Fx);
        normal_flux<double, false>(u, u, pr, fc.base, 0.0, 1.0, fc.vwy, Fy);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const double fx = Fx[c] - fvx[c], fy = Fy[c] - fvy[c];
          Fr[c] = rx * fx + ry * fy;
          Fs[c] = sx * fx + sy * fy;
        }
      }
      if constexpr (Q::TAIL) {
        wave_sync();
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          tFr[c] = tq == 0 ? Fr[c] : tFr[c];
          tFs[c] = tq == 0 ? Fs[c] : tFs[c];
        }
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        sF[(ROWC * c + ROWE * re) * FRS + rn] = Fr[c];
        sF[(16 + ROWC * c + ROWE * re) * FRS + rn] = Fs[c];
      }
      wave_sync();
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4) {
        const int s = 4 * tq + s4;
        if (s < KQ) {
          const double fr = sF[arow * FRS + 4 * s4 + acol], fs = sF[(16 + arow) * FRS + 4 * s4 + acol];
#pragma unroll
          for (int tt = 0; tt < NT; ++tt) {
            const int fo = (tt * KQ + s) * 64 + lane;
            acc[tt] = mfma(fr, G[P::OFF_WR + fo], acc[tt]);
            acc[tt] = mfma(fs, G[P::OFF_WS + fo], acc[tt]);
          }
        }
      }
      wave_sync();
    }

    if constexpr (Q::TAIL) {
      const int src = 16 * EPT + (re < EPT ? re : 0);
      double wr[NT], ws[NT];
#pragma unroll
      for (int tt = 0; tt < NT; ++tt) {
        const int fo = (tt * KQ + KQ - 1) * 64 + rn;
        wr[tt] = G[P::OFF_WR + fo];
        ws[tt] = G[P::OFF_WS + fo];
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const double fr = lane_read(tFr[c], src), fs = lane_read(tFs[c], src);
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
          acc[tt][c] = __builtin_fma(fs, ws[tt], __builtin_fma(fr, wr[tt], acc[tt][c]));
      }
    }
    if constexpr (Q::LATE) load_traces();
    // ---- K1 (and at p = 6 K0) of the tile's outputs, covered by the face pass
    double rk[NT][4], r0[NT][4];
    {
      const __amdgpu_buffer_rsrc_t rk_d = records(a != 0.0 ? K1 : Uin, e0, nel, S * 8);
      const __amdgpu_buffer_rsrc_t r0_d = records(Uin, e0, nel, S * 8);
#pragma unroll
      for (int tt = 0; tt < NT; ++tt) {
        const int n = 16 * tt + rn < Np ? 16 * tt + rn : Np - 1;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int off = (re * S + c * Np + n) * 8;
          rk[tt][c] = buf_load_f64(rk_d, off);
          r0[tt][c] = Q::OVER ? buf_load_f64(r0_d, off) : 0.0;
        }
      }
    }

    // ---- face points, one lane each
    if (ok) {
      const double* g = sGeo + pl.e * kGeoStride;
      const double nx = g[4 + 4 * pl.f], ny = g[5 + 4 * pl.f], fsc = g[6 + 4 * pl.f];
      const double up[4] = {own[0].x, own[0].y, own[1].x, own[1].y};
      const double nbu[4] = {nbt[0].x, nbt[0].y, nbt[1].x, nbt[1].y};
      double uo[4];
      ghost_state<double, false>(tag, up, up, nbu, 1, fc.vwx, fc.vwy, fc.gas, fc.base, uo);
      const double vn[4] = {0.0, tag == 0 ? 0.5 * (own[2].x - nbt[2].x) : own[2].x,
                            tag == 0 ? 0.5 * (own[2].y - nbt[2].y) : own[2].y,
                            tag == 0 ? 0.5 * (own[3].x - nbt[3].x) : own[3].x};
      const double gbar = nbt[3].y > own[3].y ? nbt[3].y : own[3].y;
      const double sigma = g[7 + 4 * pl.f] * gbar;
      const double vwn = fc.vwx * nx + fc.vwy * ny;
      const Prim<double> pp = prim_plain(up, fc.gas.gm1);
      double Fc[4];
      if (tag == 1) {
        Fc[0] = 0.0;
        Fc[1] = pp.p * nx;
        Fc[2] = pp.p * ny;
        Fc[3] = pp.p * vwn;
      } else {
        const Prim<double> po = prim_plain(uo, fc.gas.gm1);
        double FL[4], FR[4];
        normal_flux<double, false>(up, up, pp, fc.base, nx, ny, vwn, FL);
        normal_flux<double, false>(uo, uo, po, fc.base, nx, ny, vwn, FR);
        roe_flux(pp, po, FL, FR, nx, ny, vwn, fc.gas.gm1, Fc);
      }
      double w[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        w[c] = up[c] - uo[c];
        sH[(ROWC * c + ROWE * pl.e) * GRS + pl.fg] = -fsc * (Fc[c] - vn[c] + sigma * w[c]);
      }
      double qx[4], qy[4];
      viscous_transpose(tag == 1 ? gas_wall(fc.gas, fc.k_wall) : fc.gas, vstate(fc.gas, tag == 1 ? uo : up), nx,
                        ny, w, qx, qy);
      const double ce = fc.theta * (tag == 0 ? 0.5 : 1.0) * fsc;
      const double rx = g[0], ry = g[1], sx = g[2], sy = g[3];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        sQr[(ROWC * c + ROWE * pl.e) * GRS + pl.fg] = ce * (rx * qx[c] + ry * qy[c]);
        sQs[(ROWC * c + ROWE * pl.e) * GRS + pl.fg] = ce * (sx * qx[c] + sy * qy[c]);
      }
    }
    for (int i = lane; i < 48 * (GRS - NG); i += 64) {
      const int row = i / (GRS - NG);
      sH[row * GRS + NG + (i - row * (GRS - NG))] = 0.0;
    }
    wave_sync();
    load_own(tile + stride);

    // ---- lifts into the accumulator, then the RK stage
#pragma unroll
    for (int s = 0; s < KG; ++s) {
      const int ao = arow * GRS + 4 * s + acol;
      const double h = sH[ao], qr = sQr[ao], qs = sQs[ao];
#pragma unroll
      for (int tt = 0; tt < NT; ++tt) {
        const int fo = (tt * KG + s) * 64 + lane;
        acc[tt] = mfma(h, G[P::OFF_LQ + fo], acc[tt]);
        acc[tt] = mfma(qr, G[P::OFF_LRQ + fo], acc[tt]);
        acc[tt] = mfma(qs, G[P::OFF_LSQ + fo], acc[tt]);
      }
    }
    double unew[NT][4];
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) {
      const int n = 16 * tt + rn;
      if (re < nel && n < Np) {
        const int64_t base_i = (e0 + re) * S + n;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const double R = acc[tt][c];
          const int64_t idx = base_i + c * Np;
          const double kk = (a == 0.0) ? dt * R : a * rk[tt][c] + dt * R;
          K1[idx] = kk;
          const double u0 = Q::OVER ? r0[tt][c] : sU[(ROWC * c + ROWE * re) * RS + n];
          unew[tt][c] = u0 + b * kk;
          Uout[idx] = unew[tt][c];
        }
      }
    }
    if (tr_out != nullptr) {
      wave_sync();
#pragma unroll
      for (int tt = 0; tt < NT; ++tt) {
        const int n = 16 * tt + rn;
        if (re < nel && n < Np) {
#pragma unroll
          for (int c = 0; c < 4; ++c) sU[(ROWC * c + ROWE * re) * RS + n] = unew[tt][c];
        }
      }
      wave_sync();
      write_point_traces<N>(fc, pl, sU, sGeo, sF, sTab, lane, conn, nel, e0, tr_out);
    }
  }
}

template <int N, int W>
__device__ __forceinline__ void oi_lds_init(const double* __restrict__ oi, double* sTabs, double* area) {
  using Q = OITrace<N>;
  copy_values_to_lds<Q::TAB, W>(oi + Q::FIRST, sTabs);
  zero_state_pads<N>(area, threadIdx.x & 63);
  __syncthreads();
}

template <int N, int W>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(2))) void
oi_trace_stage_kernel(DeviceTables t, KernelPhysics ph, const double* __restrict__ Uin,
                      double* __restrict__ Uout, double* __restrict__ K1, double a, double b, double dt,
                      const D2* __restrict__ tr_in, D2* __restrict__ tr_out) {
  using P = OIOrder<N>;
  using Q = OITrace<N>;
  __shared__ __attribute__((aligned(16))) double sTabs[Q::TAB];
  __shared__ __attribute__((aligned(16))) double sWave[W * Q::WAVE_SZ];
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double* area = sWave + wid * Q::WAVE_SZ;
  oi_lds_init<N, W>(t.oi, sTabs, area);
  const int64_t ntiles = (t.K + P::EPT - 1) / P::EPT;
  const int xcd = blockIdx.x & 7;
  const int64_t tb = ntiles * xcd / 8, te = ntiles * (xcd + 1) / 8;
  oi_trace_tiles<N>(t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, sTabs, area,
                    tb + (int64_t)(blockIdx.x >> 3) * W + wid, te, (int64_t)(gridDim.x >> 3) * W);
}

// The traces of a given state (a call's first).
template <int N>
__global__ __launch_bounds__(256) void oi_face_trace_kernel(DeviceTables t, KernelPhysics ph,
                                                            const double* __restrict__ U,
                                                            D2* __restrict__ tr) {
  using P = OIOrder<N>;
  using Q = OITrace<N>;
  constexpr int W = 4, AREA = P::U_SZ + 64 + P::EPT * kGeoStride;
  __shared__ __attribute__((aligned(16))) double sTab[P::LDS_TAB];
  __shared__ __attribute__((aligned(16))) double sWave[W * AREA];
  copy_values_to_lds<P::LDS_TAB, W>(t.oi + P::OFF_DRSF, sTab);
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double* sU = sWave + wid * AREA;
  double* sNorm = sU + P::U_SZ;
  double* sGeo = sNorm + 64;
  __syncthreads();
  const FaceConst<double> fc = face_const<double>(ph);
  const PointLane<N> pl(lane);
  const StateRun<N> run(lane);
  const int64_t ntiles = (t.K + P::EPT - 1) / P::EPT;
  const int xcd = blockIdx.x & 7;
  const int64_t tb = ntiles * xcd / 8, te = ntiles * (xcd + 1) / 8;
  for (int64_t tile = tb + (int64_t)(blockIdx.x >> 3) * W + wid; tile < te; tile += (int64_t)(gridDim.x >> 3) * W) {
    const int64_t e0 = tile * P::EPT;
    const int nel = (int)((t.K - e0) < P::EPT ? (t.K - e0) : P::EPT);
    const __amdgpu_buffer_rsrc_t ud = records(U, e0, nel, P::S * 8);
    double ru[Q::NQ];
#pragma unroll
    for (int i = 0; i < Q::NQ; ++i) ru[i] = buf_load_f64(ud, (lane + 64 * i) * 8);
    const double rg = buf_load_f64(records(t.geo, e0, nel, kGeoStride * 8), lane * 8);
    const int conn =
        __builtin_amdgcn_raw_buffer_load_b32(records(t.conn, e0, nel, 3 * 4), (pl.e * 3 + pl.f) * 4, 0, 0);
    wave_sync();
#pragma unroll
    for (int i = 0; i < Q::NQ; ++i)
      if (lane + 64 * i < nel * P::S) sU[run.at[i]] = ru[i];
    if (lane < nel * kGeoStride) sGeo[lane] = rg;
    wave_sync();
    write_point_traces<N>(fc, pl, sU, sGeo, sNorm, sTab, lane, conn, nel, e0, tr);
  }
}

namespace {
// Waves per workgroup: at p = 4, whose 52 KB of fragments and tables leave a CU
// room for one set, eight (57.7 us a stage on 20,480 elements, with four 62);
// elsewhere four (p = 1..3: 15.9, 22.2, 27.7 us, with eight 19.3, 24.4, 30.9).
// A launch shape of two waves halves either, and so does the default where four
// waves a workgroup still leave every tile a wave of its own (p = 4, 512
// elements 13.2 instead of 17.9 us).
template <int N, int W>
int launch_oi_trace_w(const StageTuning& tune, const DeviceTables& t, const KernelPhysics& ph, const double* Uin,
                      double* Uout, double* K1, double a, double b, double dt, const void* tr_in, void* tr_out,
                      hipStream_t s, std::string& err) {
  static int cache[kMaxDev] = {0};
  const int resident = resident_blocks(oi_trace_stage_kernel<N, W>, 64 * W, cache);
  constexpr int EPT = OIOrder<N>::EPT;
  const int64_t grid = stage_grid((t.K + EPT - 1) / EPT, W, resident, tune.grid);
  hipLaunchKernelGGL((oi_trace_stage_kernel<N, W>), dim3((unsigned)grid), dim3(64 * W), 0, s, t, ph, Uin, Uout, K1,
                     a, b, dt, (const D2*)tr_in, (D2*)tr_out);
  return launch_error(err, "over-integrated trace stage launch");
}

template <int N>
int launch_oi_trace_n(const StageTuning& tune, const DeviceTables& t, const KernelPhysics& ph, const double* Uin,
                      double* Uout, double* K1, double a, double b, double dt, const void* tr_in, void* tr_out,
                      hipStream_t s, std::string& err) {
  constexpr int BIG = N == 4 ? 8 : 4;
  if ((tune.waves ? tune.waves : default_oi_trace_waves(N, t.K)) == 2)
    return launch_oi_trace_w<N, BIG / 2>(tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
  return launch_oi_trace_w<N, BIG>(tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
}

template <int N>
int launch_oi_face_n(const DeviceTables& t, const KernelPhysics& ph, const double* U, void* tr, hipStream_t s,
                     std::string& err) {
  static int cache[kMaxDev] = {0};
  const int resident = resident_blocks(oi_face_trace_kernel<N>, 256, cache);
  const int64_t grid = stage_grid((t.K + OIOrder<N>::EPT - 1) / OIOrder<N>::EPT, 4, resident, 0);
  hipLaunchKernelGGL((oi_face_trace_kernel<N>), dim3((unsigned)grid), dim3(256), 0, s, t, ph, U, (D2*)tr);
  return launch_error(err, "over-integrated face trace launch");
}
}  // namespace

int default_oi_trace_waves(int N, int64_t K) {
  const bool few = (K + OIOrder<4>::EPT - 1) / OIOrder<4>::EPT <= 4 * device_cus(current_device());
  return N == 4 && few ? 2 : 4;
}

int launch_oi_trace_stage(int N, const StageTuning& tune, const DeviceTables& t, const KernelPhysics& ph,
                          const double* Uin, double* Uout, double* K1, double a, double b, double dt,
                          const void* tr_in, void* tr_out, void* stream, std::string& err) {
  hipStream_t s = (hipStream_t)stream;
  switch (N) {
    case 1: return launch_oi_trace_n<1>(tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
    case 2: return launch_oi_trace_n<2>(tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
    case 3: return launch_oi_trace_n<3>(tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
    case 4: return launch_oi_trace_n<4>(tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
    case 5: return launch_oi_trace_n<5>(tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
    case 6: return launch_oi_trace_n<6>(tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
    default: err = "polynomial order not built"; return -5;
  }
}

int launch_oi_face_traces(int N, const DeviceTables& t, const KernelPhysics& ph, const double* U, void* tr,
                          void* stream, std::string& err) {
  hipStream_t s = (hipStream_t)stream;
  switch (N) {
    case 1: return launch_oi_face_n<1>(t, ph, U, tr, s, err);
    case 2: return launch_oi_face_n<2>(t, ph, U, tr, s, err);
    case 3: return launch_oi_face_n<3>(t, ph, U, tr, s, err);
    case 4: return launch_oi_face_n<4>(t, ph, U, tr, s, err);
    case 5: return launch_oi_face_n<5>(t, ph, U, tr, s, err);
    case 6: return launch_oi_face_n<6>(t, ph, U, tr, s, err);
    default: err = "polynomial order not built"; return -5;
  }
}

}  // namespace dgmi
