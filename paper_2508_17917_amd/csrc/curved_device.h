// The body of the curved set's stage, which the stage kernels run in their
// leading workgroups.
#pragma once

#include <hip/hip_runtime.h>

#include "stage_device.h"

namespace dgmi {

// Isoparametric elements and their face neighbours (the curved set S), in
// FP64 in every form: one element per wavefront, per-node metric terms,
// per-face-node normals and sJ, and the element's P = (M^K)^-1 M.
// With J inside the contravariant flux and sJ in the face terms, the
// strong-form residual X = -(D_r F~_r + D_s F~_s) + LIFT h + LIFT_r q_r +
// LIFT_s q_s is M times the weak form's integrals, and R = P X (on an affine
// element P = M / (J M), the stage kernel's arithmetic).  The stage kernel's
// straight tiles leave these elements unwritten, and this body reads only the
// input state and its own element's K1, so both run in the same launch: the
// stage kernel's leading workgroups take the curved set, one element per
// wave, on the SIMDs beside the straight tiles.  lds: the wave's area,
// curved_lds_doubles(N) doubles.
//
// A curved wave is one chain of dependent phases, the longest in a launch, so
// what it waits for is loaded ahead: the three neighbours' states with the own
// one (in LDS until the face terms take their place), the operators' rows eight
// at a time, K1 before the product with P.
constexpr int curved_face_doubles(int N) {  // neighbours' states, later the face terms
  return 36 * (N + 1) > 6 * (N + 1) * (N + 2) ? 36 * (N + 1) : 6 * (N + 1) * (N + 2);
}
constexpr int curved_lds_doubles(int N) {
  return 29 * ((N + 1) * (N + 2) / 2) + curved_face_doubles(N) + 3 * (N + 1);
}
// workgroups of W waves that take the curved set, a multiple of 8 (so the
// straight tiles' workgroups keep their XCD numbering)
__host__ __device__ inline int curved_workgroups(int ncurved, int W) {
  return ncurved > 0 ? ((ncurved + W - 1) / W + 7) / 8 * 8 : 0;
}
template <int N>
__device__ __forceinline__ void curved_element(const DeviceTables& t, const KernelPhysics& ph,
                                               const double* __restrict__ Uin,
                                               double* __restrict__ Uout,
                                               double* __restrict__ K1, double a, double b,
                                               double dt, int rhs_only, int slot, double* lds) {
  constexpr int Np = (N + 1) * (N + 2) / 2, Nfp = N + 1, NFN = 3 * Nfp, S = 4 * Np;
  double* sU = lds;
  double* sGx = sU + S;
  double* sGy = sGx + S;
  double* sFr = sGy + S;
  double* sFs = sFr + S;
  double* sX = sFs + S;
  double* sNd = sX + S;
  double* sH = sNd + 5 * Np;
  double* sQr = sH + 4 * NFN;
  double* sQs = sQr + 4 * NFN;
  double* sNb = sH;  // [face][S]
  double* sNorm = sH + curved_face_doubles(N);
  static_assert(6 * S + 5 * Np + curved_face_doubles(N) + NFN == curved_lds_doubles(N), "curved LDS layout");
  const int lane = threadIdx.x & 63;
  const int64_t k = t.celem[slot];
  const double* Dr = t.ops;
  const double* Ds = t.ops + Np * Np;
  const double* LIFT = t.ops + 2 * Np * Np;
  const double* LIFTr = LIFT + Np * NFN;
  const double* LIFTs = LIFTr + Np * NFN;
  const double* nd = t.cnode + (int64_t)slot * 5 * Np;
  const double* fc = t.cface + (int64_t)slot * 3 * NFN;
  Gas<double> gas;
  gas.gamma = ph.gamma;
  gas.gm1 = ph.gm1;
  gas.igm1 = ph.igm1;
  gas.mu = ph.mu;
  gas.k = ph.k;
  Base<double> base;
  base.rho = ph.U_inf[0];
  base.mx = ph.U_inf[1];
  base.my = ph.U_inf[2];
  base.E = ph.U_inf[3];
  base.p = ph.p_inf;
  base.ux = ph.u_inf;
  base.uy = ph.v_inf;
  const double vwx = ph.vw[0], vwy = ph.vw[1];

  {
    // own state, node metrics and the neighbours' states (a boundary face's is
    // the element's own, unused), every load in flight
    constexpr int LU = (S + 63) / 64, LN = (5 * Np + 63) / 64, LB = (3 * S + 63) / 64;
    double ru[LU], rn[LN], rb[LB];
#pragma unroll
    for (int q = 0; q < LB; ++q) {
      const int i = lane + 64 * q < 3 * S ? lane + 64 * q : 0, fb = i / S;
      rb[q] = Uin[(int64_t)(t.conn[k * 3 + fb] >> 4) * S + (i - fb * S)];
    }
#pragma unroll
    for (int q = 0; q < LU; ++q) ru[q] = Uin[k * S + (lane + 64 * q < S ? lane + 64 * q : 0)];
#pragma unroll
    for (int q = 0; q < LN; ++q) rn[q] = nd[lane + 64 * q < 5 * Np ? lane + 64 * q : 0];
#pragma unroll
    for (int q = 0; q < LU; ++q)
      if (lane + 64 * q < S) sU[lane + 64 * q] = ru[q];
#pragma unroll
    for (int q = 0; q < LN; ++q)
      if (lane + 64 * q < 5 * Np) sNd[lane + 64 * q] = rn[q];
#pragma unroll
    for (int q = 0; q < LB; ++q)
      if (lane + 64 * q < 3 * S) sNb[lane + 64 * q] = rb[q];
  }
  wave_sync();
  // gradient at the nodes with each node's metric terms
  #pragma unroll 1
  for (int i = lane; i < S; i += 64) {
    const int c = i / Np, n = i - c * Np;
    double ur = 0.0, us = 0.0;
    #pragma unroll 8
    for (int m = 0; m < Np; ++m) {
      ur += Dr[n * Np + m] * sU[c * Np + m];
      us += Ds[n * Np + m] * sU[c * Np + m];
    }
    sGx[i] = sNd[n] * ur + sNd[2 * Np + n] * us;
    sGy[i] = sNd[Np + n] * ur + sNd[3 * Np + n] * us;
  }
  wave_sync();
  // total flux at the nodes, contravariant with J
  #pragma unroll 1
  for (int n = lane; n < Np; n += 64) {
    double u[4], gx[4], gy[4];
    for (int c = 0; c < 4; ++c) {
      u[c] = sU[c * Np + n];
      gx[c] = sGx[c * Np + n];
      gy[c] = sGy[c * Np + n];
    }
    double fvx[4], fvy[4], Fx[4], Fy[4];
    viscous_flux(gas, vstate(gas, u), gx, gy, fvx, fvy);
    const Prim<double> pr = prim_plain(u, gas.gm1);
    normal_flux_plain(u, pr, 1.0, 0.0, vwx, Fx);
    normal_flux_plain(u, pr, 0.0, 1.0, vwy, Fy);
    const double rx = sNd[n], ry = sNd[Np + n], sx = sNd[2 * Np + n], sy = sNd[3 * Np + n];
    const double J = sNd[4 * Np + n];
    for (int c = 0; c < 4; ++c) {
      const double fx = Fx[c] - fvx[c], fy = Fy[c] - fvy[c];
      sFr[c * Np + n] = J * (rx * fx + ry * fy);
      sFs[c * Np + n] = J * (sx * fx + sy * fy);
    }
  }
  wave_sync();
  // face nodes, one lane each: traces, ghosts, norms, the other side's
  // gradient (with that element's metric terms at its node), viscous mean
  const bool fl = lane < NFN;
  const int l = fl ? lane : 0;
  const int f = l / Nfp, j = l - f * Nfp;
  const int n = face_node<N>(f, j);
  const int conn = t.conn[k * 3 + f];
  const int tag = conn & 3, nf = (conn >> 2) & 3;
  const int64_t kn = conn >> 4;
  const double nx = fc[l], ny = fc[NFN + l], sJ = fc[2 * NFN + l];
  double up[4] = {0.0, 0.0, 0.0, 0.0}, uo[4] = {0.0, 0.0, 0.0, 0.0};
  double vn[4] = {0.0, 0.0, 0.0, 0.0};
  VState<double> sp = {}, so = {};
  if (fl) {
    double gxp[4], gyp[4], gxm[4], gym[4];
    for (int c = 0; c < 4; ++c) {
      up[c] = sU[c * Np + n];
      gxp[c] = sGx[c * Np + n];
      gyp[c] = sGy[c * Np + n];
      gxm[c] = gxp[c];
      gym[c] = gyp[c];
    }
    if (tag == 0) {
      const int n2 = face_node<N>(nf, Nfp - 1 - j);
      const double* Un = sNb + f * S;
      double ur[4] = {0, 0, 0, 0}, us[4] = {0, 0, 0, 0};
      #pragma unroll 8
      for (int m = 0; m < Np; ++m) {
        const double dr = Dr[n2 * Np + m], ds = Ds[n2 * Np + m];
        for (int c = 0; c < 4; ++c) {
          ur[c] += dr * Un[c * Np + m];
          us[c] += ds * Un[c * Np + m];
        }
      }
      const int cs = t.cslot[kn];
      double rx, ry, sx, sy;
      if (cs >= 0) {
        const double* nd2 = t.cnode + (int64_t)cs * 5 * Np;
        rx = nd2[n2];
        ry = nd2[Np + n2];
        sx = nd2[2 * Np + n2];
        sy = nd2[3 * Np + n2];
      } else {
        const double* g2 = t.geo + kn * kGeoStride;
        rx = g2[0];
        ry = g2[1];
        sx = g2[2];
        sy = g2[3];
      }
      for (int c = 0; c < 4; ++c) {
        uo[c] = Un[c * Np + n2];
        gxm[c] = rx * ur[c] + sx * us[c];
        gym[c] = ry * ur[c] + sy * us[c];
      }
    } else {
      // wall or far field: the ghost (no neighbour value is read)
      ghost_state<double, false>(tag, up, up, sU + n, Np, vwx, vwy, gas, base, uo);
    }
    sp = vstate(gas, up);
    so = vstate(gas, uo);
    const double a1 = normal_diffusion_norm(gas, sp, nx, ny);
    const double a2 = normal_diffusion_norm(gas, so, nx, ny);
    sNorm[l] = a1 > a2 ? a1 : a2;
    if (tag == 1) {
      // wall: G(U^b) grad U+ (conduction as the wall flux mode sets it)
      viscous_normal_flux(gas_wall(gas, ph.k_wall), so, gxp, gyp, nx, ny, vn);
    } else {
      viscous_normal_flux(gas, sp, gxp, gyp, nx, ny, vn);
      if (tag == 0) {
        double vm[4];
        viscous_normal_flux(gas, so, gxm, gym, nx, ny, vm);
        for (int c = 0; c < 4; ++c) vn[c] = 0.5 * (vn[c] + vm[c]);
      }
    }
  }
  wave_sync();
  if (fl) {
    double gbar = 0.0;
    #pragma unroll 1
    for (int jj = 0; jj < Nfp; ++jj) gbar = sNorm[f * Nfp + jj] > gbar ? sNorm[f * Nfp + jj] : gbar;
    const double sigma = t.geo[k * kGeoStride + 7 + 4 * f] * gbar;
    const double vwn = vwx * nx + vwy * ny;
    const Prim<double> pp = prim_plain(up, gas.gm1);
    double Fc[4];
    if (tag == 1) {
      Fc[0] = 0.0;
      Fc[1] = pp.p * nx;
      Fc[2] = pp.p * ny;
      Fc[3] = pp.p * vwn;
    } else {
      const Prim<double> po = prim_plain(uo, gas.gm1);
      double FL[4], FR[4];
      normal_flux_plain(up, pp, nx, ny, vwn, FL);
      normal_flux_plain(uo, po, nx, ny, vwn, FR);
      roe_flux(pp, po, FL, FR, nx, ny, vwn, gas.gm1, Fc);
    }
    // sJ times the own normal flux, from the contravariant flux (J inside):
    // face 0: -Fs, face 1: Fr + Fs, face 2: -Fr
    const double cfr = f == 0 ? 0.0 : (f == 1 ? 1.0 : -1.0);
    const double cfs = f == 2 ? 0.0 : (f == 1 ? 1.0 : -1.0);
    double w[4];
    for (int c = 0; c < 4; ++c) {
      w[c] = up[c] - uo[c];
      const double own = cfr * sFr[c * Np + n] + cfs * sFs[c * Np + n];
      sH[c * NFN + l] = own - sJ * (Fc[c] - vn[c] + sigma * w[c]);
    }
    double qx[4], qy[4];
    viscous_transpose(tag == 1 ? gas_wall(gas, ph.k_wall) : gas, tag == 1 ? so : sp, nx, ny, w, qx, qy);
    const double ce = ph.theta * (tag == 0 ? 0.5 : 1.0) * sJ;
    const double rx = sNd[n], ry = sNd[Np + n], sx = sNd[2 * Np + n], sy = sNd[3 * Np + n];
    for (int c = 0; c < 4; ++c) {
      sQr[c * NFN + l] = ce * (rx * qx[c] + ry * qy[c]);
      sQs[c * NFN + l] = ce * (sx * qx[c] + sy * qy[c]);
    }
  }
  wave_sync();
  // strong-form residual, then R = P X and the stage
  #pragma unroll 1
  for (int i = lane; i < S; i += 64) {
    const int c = i / Np, m0 = i - c * Np;
    double x = 0.0;
    #pragma unroll 8
    for (int m = 0; m < Np; ++m) x -= Dr[m0 * Np + m] * sFr[c * Np + m] + Ds[m0 * Np + m] * sFs[c * Np + m];
    #pragma unroll 6
    for (int q = 0; q < NFN; ++q)
      x += LIFT[m0 * NFN + q] * sH[c * NFN + q] + LIFTr[m0 * NFN + q] * sQr[c * NFN + q] +
           LIFTs[m0 * NFN + q] * sQs[c * NFN + q];
    sX[i] = x;
  }
  wave_sync();
  const double* P = t.cP + (int64_t)slot * Np * Np;
  #pragma unroll 1
  for (int i = lane; i < S; i += 64) {
    const int c = i / Np, m0 = i - c * Np;
    double R = 0.0;
    const int64_t idx = k * S + i;
    const double k1 = a != 0.0 ? K1[idx] : 0.0;
    #pragma unroll 8
    for (int m = 0; m < Np; ++m) R += P[m0 * Np + m] * sX[c * Np + m];
    if (rhs_only) {
      K1[idx] = R;
    } else {
      const double kk = (a != 0.0) ? a * k1 + dt * R : dt * R;
      K1[idx] = kk;
      sU[i] += b * kk;  // the new state, for a caller that needs it
      Uout[idx] = sU[i];
    }
  }
}

}  // namespace dgmi
