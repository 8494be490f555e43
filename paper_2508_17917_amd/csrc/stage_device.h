// Device pieces shared by the stage kernels (kernels.hip, trace.hip): the per-order
// layout constants, matrix-core and descriptor helpers, ghost states, the wall
// force, and the host-side launch shape.
#pragma once

#include <hip/hip_runtime.h>

#include <string>

#include "dg_internal.h"
#include "dg_physics.h"

namespace dgmi {

// Real types of the right-hand side: double, float, or float with the
// operator products on the bfloat16 matrix cores (FP32 accumulation).
struct bf16ops {};
template <typename X>
struct Real {
  typedef X type;
  static constexpr bool bf = false;
};
template <>
struct Real<bf16ops> {
  typedef float type;
  static constexpr bool bf = true;
};

template <int N, typename X>
struct Order {
  typedef typename Real<X>::type T;
  static constexpr bool BF = Real<X>::bf;
  static constexpr int Np = (N + 1) * (N + 2) / 2;
  static constexpr int Nfp = N + 1;
  static constexpr int NF = 3 * (N + 1);
  static constexpr int S = 4 * Np;               // values per element state
  static constexpr int NT = (Np + 15) / 16;      // 16-node output tiles
  static constexpr int KS = (Np + 3) / 4;        // k-steps over volume nodes
  static constexpr int KF = (NF + 3) / 4;        // k-steps over face nodes
  static constexpr int KS16 = (Np + 15) / 16;    // bfloat16 k-steps (16 deep)
  static constexpr int KF16 = (NF + 15) / 16;
  // padded LDS rows (odd: no bank aliasing), long enough for the k-steps
  static constexpr int RS = (BF && 16 * KS16 > 4 * KS ? 16 * KS16 : 4 * KS) + 1;
  static constexpr int HRS = (BF && 16 * KF16 > 4 * KF ? 16 * KF16 : 4 * KF) + 1;
  static constexpr int EPT = elements_per_tile(N);  // elements per tile (4 slots)
  static constexpr int FIT = (EPT * NF + 63) / 64;  // face items per lane
  // the volume flux in one pass over (element, node) pairs packed onto the
  // lanes, where they fit 64 lanes but the matrix-core layout (16 node
  // columns x 4 element slots per output tile) needs several tiles: p = 5
  // (3 x 21 of 64 lanes in one pass instead of 63 of 128 in two)
  static constexpr bool PACK = (EPT * Np <= 64) && (NT > 1);
  // default waves per workgroup (each wave owns its own tiles; the workgroup
  // shares the operator fragments)
  // (4 measured fastest for every order and form on MI355X: the fragments
  // are shared by more waves, and at p >= 5 in FP64 LDS and registers allow
  // one workgroup per CU either way)
  static constexpr int WAVES = 4;
  // waves per SIMD the register allocation must allow: 3 for FP32 at p <= 4
  // (a few spills, measured faster than 2 and than 4), else 2
  static constexpr int MIN_WAVES_EU = (sizeof(T) == 4 && N <= 4) ? 3 : 2;
  // the next tile's own data issued before the face pass where the
  // registers allow (K1 / K0 of the tile always are)
  static constexpr bool EARLY_OWN = N <= 4;
  // per-wave LDS (elements of T)
  static constexpr int U_SZ = 16 * RS;           // own state
  static constexpr int F_SZ = 32 * RS;           // contravariant flux Fr rows | Fs rows
  static constexpr int N_SZ = 12 * S;            // neighbour states [e][f][c][n]
  static constexpr int H_SZ = 48 * HRS;          // face terms h | qr | qs
  static constexpr int X_SZ = N_SZ > H_SZ ? N_SZ : H_SZ;
  static constexpr int NORM_SZ = 4 * NF;
  static constexpr int WAVE_SZ = U_SZ + F_SZ + X_SZ + NORM_SZ + 64 + 48;
  // operator fragments (per workgroup)
  // one Dr-type / LIFT-type fragment set, in elements of T (bfloat16: four
  // values per lane, i.e. two floats' worth)
  static constexpr int FD = BF ? NT * KS16 * 64 * 2 : NT * KS * 64;
  static constexpr int FL = BF ? NT * KF16 * 64 * 2 : NT * KF * 64;
  static constexpr int FRAG_SZ = 2 * FD + 3 * FL;
  // matrix-core row of (field c, element e): the FP64 instruction returns rows
  // l/16 + 4v to lane l, the FP32 one rows 4(l/16) + v; either way lane l ends
  // up with element l/16 and field v
  static constexpr int ROWC = sizeof(T) == 8 ? 4 : 1;
  static constexpr int ROWE = sizeof(T) == 8 ? 1 : 4;
};

// Fourth word of a raw buffer descriptor on gfx9-family devices: 32-bit data
// format (untyped loads need a valid one), no swizzle, no index stride.
constexpr int kBufferWord3 = 0x00020000;

// A raw buffer descriptor over n consecutive records of `bytes_each` bytes
// starting at record r0 of the array at p (built on the scalar unit when its
// arguments are uniform).  Accesses past the n records read 0 and write
// nothing (the hardware's range check), so n <= 0 gives an empty range.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t records(const void* p, int64_t r0, int64_t n,
                                                          int bytes_each) {
  const int bytes = n > 0 ? (int)(n * bytes_each) : 0;
  return __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p + r0 * bytes_each), (short)0, bytes,
                                           kBufferWord3);
}
__device__ __forceinline__ double buf_load_f64(__amdgpu_buffer_rsrc_t r, int byte_off) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, byte_off, 0, 0));
}

// Copy N values from global memory to LDS by the 64 W threads of a workgroup,
// 16 bytes a lane with every load in flight before the first store (one load
// and one store at a time take a memory round trip per iteration: 16.3 instead
// of 15.8 us a stage at p = 4 FP32 on 20,480 elements, at p = 5 30.3 instead of
// 28.2, over-integrated p = 4 56.3 instead of 54.0).
// Both arrays 16-byte aligned, N * sizeof(T) a multiple of 16.
template <int N, int W, typename T>
__device__ __forceinline__ void copy_to_lds(const T* __restrict__ src, T* dst) {
  static_assert((N * sizeof(T)) % 16 == 0, "whole 16-byte vectors");
  constexpr int NV = (int)(N * sizeof(T) / 16), PER = (NV + 64 * W - 1) / (64 * W);
  uint4 v[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int i = (int)threadIdx.x + 64 * W * q;
    v[q] = ((const uint4*)src)[i < NV ? i : NV - 1];
  }
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int i = (int)threadIdx.x + 64 * W * q;
    if (i < NV) ((uint4*)dst)[i] = v[q];
  }
}

// The same for any count of doubles (the last one by itself where it is odd).
template <int N, int W>
__device__ __forceinline__ void copy_values_to_lds(const double* __restrict__ src, double* dst) {
  copy_to_lds<N / 2 * 2, W>(src, dst);
  if (N % 2 != 0 && threadIdx.x == 0) dst[N - 1] = src[N - 1];
}

// Node index of face node j (counter-clockwise) on face f; rows of the node
// numbering start at i(N+1) - i(i-1)/2.
template <int N>
__device__ __forceinline__ int face_node(int f, int j) {
  if (f == 0) return j;
  if (f == 1) return j * (N + 1) - j * (j - 1) / 2 + (N - j);
  int i = N - j;
  return i * (N + 1) - i * (i - 1) / 2;
}

template <typename T>
struct Vec4 {
  typedef T type __attribute__((ext_vector_type(4)));
};

// D += A B for A 16x4, B 4x16, D 16x16 on the matrix cores.  Lane l supplies
// A[l%16][l/16] and B[l/16][l%16]; it holds D[l/16 + 4v][l%16] (FP64) or
// D[4(l/16) + v][l%16] (FP32), v = 0..3.
__device__ __forceinline__ Vec4<double>::type mfma(double a, double b, Vec4<double>::type c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ Vec4<float>::type mfma(float a, float b, Vec4<float>::type c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// bfloat16 operands (16x16x16, FP32 accumulation): lane l supplies
// A[l%16][4(l/16) + j] and B[4(l/16) + j][l%16]; the result layout is that of
// the FP32 instruction.
typedef short bf16x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ unsigned short to_bf16(float f) {
  unsigned u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);  // round to nearest, ties to even
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ bf16x4_t bf16_row(const float* p) {
  return bf16x4_t{(short)to_bf16(p[0]), (short)to_bf16(p[1]), (short)to_bf16(p[2]),
                  (short)to_bf16(p[3])};
}
__device__ __forceinline__ bf16x4_t bf16_frag(const float* frag, int lane) {
  const uint2 w = ((const uint2*)frag)[lane];
  return bf16x4_t{(short)(w.x & 0xffff), (short)(w.x >> 16), (short)(w.y & 0xffff),
                  (short)(w.y >> 16)};
}
__device__ __forceinline__ Vec4<float>::type mfma_bf16(bf16x4_t a, bf16x4_t b,
                                                       Vec4<float>::type c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// LDS ordering among the lanes of one wavefront (no workgroup barrier).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ double lane_read(double v, int src) {
  int lo = __builtin_amdgcn_ds_bpermute(src << 2, __double2loint(v));
  int hi = __builtin_amdgcn_ds_bpermute(src << 2, __double2hiint(v));
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float lane_read(float v, int src) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(src << 2, __float_as_int(v)));
}

template <typename T, bool PERT>
__device__ __forceinline__ void full_state(const T u[4], const Base<T>& b, T uf[4]) {
  if (PERT) {
    uf[0] = b.rho + u[0];
    uf[1] = b.mx + u[1];
    uf[2] = b.my + u[2];
    uf[3] = b.E + u[3];
  } else {
#pragma unroll
    for (int c = 0; c < 4; ++c) uf[c] = u[c];
  }
}

template <typename T, bool PERT>
__device__ __forceinline__ Prim<T> prim_of(const T uf[4], const T u[4], const Base<T>& b, T gm1) {
  return PERT ? prim_pert(uf, u, b, gm1) : prim_plain(uf, gm1);
}

template <typename T, bool PERT>
__device__ __forceinline__ void normal_flux(const T uf[4], const T u[4], const Prim<T>& s,
                                            const Base<T>& b, T nx, T ny, T vwn, T F[4]) {
  if (PERT)
    normal_flux_pert(u, s, b, nx, ny, vwn, F);
  else
    normal_flux_plain(uf, s, nx, ny, vwn, F);
}

// Value of the state on the other side of a face node (in what the kernel
// stores: the state, or its perturbation from U_inf): the neighbour's trace
// (interior, periodic), the moving adiabatic wall's ghost Q^b = [rho+, v_w,
// p+], or the far field U_inf (Sec. 2.2.4).  nb points at the neighbour's
// node, stride Np; up is the own value, upf the own full state.
template <typename T, bool PERT>
__device__ __forceinline__ void ghost_state(int tag, const T up[4], const T upf[4], const T* nb,
                                            int Np, T vwx, T vwy, const Gas<T>& gas,
                                            const Base<T>& b, T uo[4]) {
  if (tag == 0) {
#pragma unroll
    for (int c = 0; c < 4; ++c) uo[c] = nb[c * Np];
  } else if (tag == 1) {
    const T rho = upf[0];
    const T kw = T(0.5) * rho * (vwx * vwx + vwy * vwy);
    const Prim<T> s = prim_of<T, PERT>(upf, up, b, gas.gm1);
    if (!PERT) {
      uo[0] = rho;
      uo[1] = rho * vwx;
      uo[2] = rho * vwy;
      uo[3] = s.p * gas.igm1 + kw;
    } else {
      uo[0] = up[0];
      uo[1] = rho * vwx - b.mx;
      uo[2] = rho * vwy - b.my;
      // eps_b - eps_inf = p'/(gamma-1) + rho |v_w|^2/2 - rho_inf |u_inf|^2/2
      uo[3] = s.jp * gas.igm1 + kw - T(0.5) * (b.mx * b.ux + b.my * b.uy);
    }
  } else {
    if (PERT) {
#pragma unroll
      for (int c = 0; c < 4; ++c) uo[c] = T(0);
    } else {
      uo[0] = b.rho;
      uo[1] = b.mx;
      uo[2] = b.my;
      uo[3] = b.E;
    }
  }
}

template <typename X>
__device__ __forceinline__ const typename Real<X>::type* frag_of(const DeviceTables& t);
template <>
__device__ __forceinline__ const double* frag_of<double>(const DeviceTables& t) {
  return t.frag;
}
template <>
__device__ __forceinline__ const float* frag_of<float>(const DeviceTables& t) {
  return t.frag32;
}
// bfloat16 fragments, moved as 32-bit words (never used as floats)
template <>
__device__ __forceinline__ const float* frag_of<bf16ops>(const DeviceTables& t) {
  return (const float*)t.frag16;
}

// K1 (and, in the perturbation form, K0) of output lane (element slot re,
// nodes 16 tt + rn) of the tile at element e0, into registers; returns whether
// the element is outside the curved set.  K1 is read only when the stage uses
// it (a != 0, not a bare right-hand side): otherwise the load reads the
// element's own state, which the tile has just brought into the cache, and is
// not used.
template <int N, typename X, bool PERT>
__device__ __forceinline__ bool load_k(const DeviceTables& t, const double* __restrict__ Uin,
                                       const double* __restrict__ K1, double a, int rhs_only,
                                       int64_t e0, int nel, int re, int rn,
                                       double (&rk)[Order<N, X>::NT][4],
                                       double (&r0)[Order<N, X>::NT][4]) {
  using O = Order<N, X>;
  constexpr int Np = O::Np, S = O::S;
  // descriptors over the tile's elements: the lane's offsets are constants
  const __amdgpu_buffer_rsrc_t rk_d = records((a != 0.0 && !rhs_only) ? K1 : Uin, e0, nel, S * 8);
  const __amdgpu_buffer_rsrc_t r0_d = records(Uin, e0, nel, S * 8);
#pragma unroll
  for (int tt = 0; tt < O::NT; ++tt) {
    const int n = 16 * tt + rn < Np ? 16 * tt + rn : Np - 1;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int off = (re * S + c * Np + n) * 8;
      rk[tt][c] = buf_load_f64(rk_d, off);
      r0[tt][c] = PERT ? buf_load_f64(r0_d, off) : 0.0;
    }
  }
  const int64_t ke = (e0 + re) < t.K ? (e0 + re) : t.K - 1;
  return t.cslot == nullptr || t.cslot[ke] < 0;
}

// The wall force (the traction of eq. force_integral: pressure minus the
// viscous normal stress, and its moment about the origin) at wall face node i
// (node i % Nfp of face t.wall[i / Nfp]) of the state U: the node's quadrature
// weight times sJ times (tx, ty, x ty - y tx), in FP64 in every form.  UNR:
// the unroll factor of the node's derivative loop (the same operations in the
// same order whatever it is; a smaller one holds fewer registers where the
// force runs inside the stage kernel).
constexpr int kForceThreads = 64;
template <int N, int UNR = (N + 1) * (N + 2) / 2>
__device__ __forceinline__ void wall_node_force(const DeviceTables& t, const KernelPhysics& ph,
                                                const double* __restrict__ U, int i, double& fx,
                                                double& fy, double& mz) {
  using O = Order<N, double>;
  constexpr int Np = O::Np, Nfp = O::Nfp, S = 4 * Np;
  Gas<double> gas;
  gas.gamma = ph.gamma;
  gas.gm1 = ph.gamma - 1.0;
  gas.igm1 = 1.0 / (ph.gamma - 1.0);
  gas.mu = ph.mu;
  gas.k = ph.gamma / ph.Pr;
  const double* Dr = t.ops;
  const double* Ds = t.ops + Np * Np;
  const double* wface = t.ops + 2 * Np * Np + 3 * Np * 3 * Nfp;
  const int wf = t.wall[i / Nfp];
  const int j = i % Nfp;
  const int64_t k = wf / 3;
  const int f = wf % 3;
  const int n = face_node<N>(f, j);
  const double* Uk = U + k * S;
  const double* g = t.geo + k * kGeoStride;
  // metric terms at the node, normal and sJ at the face node: per node on
  // the elements of the curved set, the element's constants elsewhere
  double rx = g[0], ry = g[1], sx = g[2], sy = g[3];
  double nx = g[4 + 4 * f], ny = g[5 + 4 * f];
  double sJ = g[6 + 4 * f] / (g[0] * g[3] - g[1] * g[2]);  // Fscale * J
  const int cs = t.cslot ? t.cslot[k] : -1;
  if (cs >= 0) {
    const double* nd = t.cnode + (int64_t)cs * 5 * Np;
    const double* fc = t.cface + (int64_t)cs * 9 * Nfp;
    rx = nd[n];
    ry = nd[Np + n];
    sx = nd[2 * Np + n];
    sy = nd[3 * Np + n];
    nx = fc[f * Nfp + j];
    ny = fc[3 * Nfp + f * Nfp + j];
    sJ = fc[6 * Nfp + f * Nfp + j];
  }
  double ur[4] = {0, 0, 0, 0}, us[4] = {0, 0, 0, 0};
#pragma unroll UNR
  for (int m = 0; m < Np; ++m) {
    const double dr = Dr[n * Np + m], ds = Ds[n * Np + m];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      ur[c] += dr * Uk[c * Np + m];
      us[c] += ds * Uk[c * Np + m];
    }
  }
  double Up[4], dx[4], dy[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    Up[c] = Uk[c * Np + n];
    dx[c] = rx * ur[c] + sx * us[c];
    dy[c] = ry * ur[c] + sy * us[c];
  }
  const double p = gas.gm1 * (Up[3] - 0.5 * (Up[1] * Up[1] + Up[2] * Up[2]) / Up[0]);
  double Ub[4] = {Up[0], Up[0] * ph.vw[0], Up[0] * ph.vw[1],
                  p * gas.igm1 + 0.5 * Up[0] * (ph.vw[0] * ph.vw[0] + ph.vw[1] * ph.vw[1])};
  double vx[4], vy[4];
  viscous_flux(gas, vstate(gas, Ub), dx, dy, vx, vy);
  const double w = wface[f * Nfp + j] * sJ;
  const double tx = p * nx - (vx[1] * nx + vy[1] * ny);
  const double ty = p * ny - (vx[2] * nx + vy[2] * ny);
  const double xw = t.wall_xy[2 * i], yw = t.wall_xy[2 * i + 1];
  fx = w * tx;
  fy = w * ty;
  mz = w * (xw * ty - yw * tx);
}

// The force from the nblk partials an earlier launch wrote, in block order:
// lane c < 3 writes component c (eight loads in flight at a time, the sum
// itself in block order, as the ticket's last wave adds them).
__device__ __forceinline__ void force_sum(const double* __restrict__ part, double* out,
                                          unsigned nblk) {
  const int lane = threadIdx.x & 63;
  if (lane < 3) {
    double sum = 0.0;
    for (unsigned b = 0; b < nblk; b += 8) {
      double v[8];
#pragma unroll
      for (unsigned q = 0; q < 8; ++q) v[q] = b + q < nblk ? part[3 * (b + q) + lane] : 0.0;
#pragma unroll
      for (unsigned q = 0; q < 8; ++q)
        if (b + q < nblk) sum += v[q];
    }
    out[lane] = sum;
  }
}

// One wave's share of the wall force: nodes 64 blk .. 64 blk + 63 of the nblk
// blocks of 64 that cover the wall face nodes, reduced by a fixed shuffle
// tree into partial blk.  With TICKET the last wave to finish (an atomic
// ticket) sums the partials in block order into out[0..2] and resets the
// ticket; without, the partials are left for a later launch to sum (the
// ticket's device-scope fences write back and invalidate the L2 of the
// wave's XCD, and its chain of round trips outlasts a stage launch's first
// tiles).  The order of every sum is fixed by the wall face list alone, so
// the total does not depend on which waves ran the blocks or in which launch.
template <int N, int UNR = (N + 1) * (N + 2) / 2, bool TICKET = true>
__device__ __forceinline__ void force_wave(const DeviceTables& t, const KernelPhysics& ph,
                                           const double* __restrict__ U, double* __restrict__ out,
                                           unsigned blk, unsigned nblk) {
  const int lane = threadIdx.x & 63;
  double fx = 0.0, fy = 0.0, mz = 0.0;
  const int i = (int)blk * kForceThreads + lane;
  if (i < t.nwall * (N + 1)) wall_node_force<N, UNR>(t, ph, U, i, fx, fy, mz);
  for (int o = 32; o > 0; o >>= 1) {
    fx += __shfl_down(fx, o, 64);
    fy += __shfl_down(fy, o, 64);
    mz += __shfl_down(mz, o, 64);
  }
  if (lane == 0) {
    t.force_part[3 * blk + 0] = fx;
    t.force_part[3 * blk + 1] = fy;
    t.force_part[3 * blk + 2] = mz;
  }
  if constexpr (!TICKET) return;
  unsigned last = 0;
  if (lane == 0) {
    __threadfence();
    last = atomicAdd(t.force_ticket, 1u) == nblk - 1;
  }
  last = __shfl(last, 0, 64);
  if (last && lane < 3) {
    __threadfence();
    const volatile double* part = t.force_part;
    double sum = 0.0;
    for (unsigned b = 0; b < nblk; ++b) sum += part[3 * b + lane];
    out[lane] = sum;
    if (lane == 0) atomicExch(t.force_ticket, 0u);
  }
}

// Sizes of the over-integrated stage of order N and the layout of its operator
// fragments and face-point tables (the order the host packs them in).
template <int N>
struct OIOrder {
  using O = Order<N, double>;
  static constexpr int Np = O::Np, Nfp = O::Nfp, S = O::S, NT = O::NT, KS = O::KS, RS = O::RS;
  static constexpr int q = oi_points(N), Nq = q * q, NG = 3 * q;
  static constexpr int NQT = (Nq + 15) / 16;   // 16-point chunks of the element rule
  static constexpr int KQ = (Nq + 3) / 4;      // k-steps over the element points
  static constexpr int KG = (NG + 3) / 4;      // k-steps over the face points
  static constexpr int EPT = (64 / NG) < 4 ? ((64 / NG) > 0 ? 64 / NG : 1) : 4;
  static constexpr int FRS = 17;               // padded LDS row of one flux chunk
  static constexpr int GRS = 4 * KG + 1;       // padded LDS row of the face terms
  static constexpr int U_SZ = 16 * RS, F_SZ = 32 * FRS;
  static constexpr int N_SZ = 12 * S, H_SZ = 48 * GRS;
  static constexpr int X_SZ = N_SZ > H_SZ ? N_SZ : H_SZ;
  static constexpr int NORM_SZ = 4 * NG, VN_SZ = 16 * NG;
  static constexpr int WAVE_SZ = (U_SZ + F_SZ + X_SZ + NORM_SZ + VN_SZ + 64 + 48 + 3) / 4 * 4;
  // global fragment offsets (doubles), in the order the host packs them
  static constexpr int FI = NQT * KS * 64, FW = NT * KQ * 64, FL = NT * KG * 64;
  static constexpr int OFF_IQ = 0, OFF_DRQ = FI, OFF_DSQ = 2 * FI, OFF_WR = 3 * FI,
                       OFF_WS = 3 * FI + FW, OFF_LQ = 3 * FI + 2 * FW, OFF_LRQ = OFF_LQ + FL,
                       OFF_LSQ = OFF_LQ + 2 * FL, OFF_DRSF = OFF_LQ + 3 * FL,
                       OFF_IF1 = OFF_DRSF + 2 * NG * Np, TOTAL = OFF_IF1 + q * Nfp;
  static constexpr int LDS_TAB = 2 * NG * Np + q * Nfp;  // face-point tables in LDS
};

// workgroups of W waves for the wall force in a stage launch: one wave per 64
// wall face nodes (the partials of the launch's input state), then the wave
// that sums a previous launch's partials; a multiple of 8, or none
__host__ __device__ inline int force_workgroups(const DeviceTables& t, int Nfp, int W) {
  const int nblk = (t.nwall * Nfp + kForceThreads - 1) / kForceThreads;
  if (nblk <= 0 || (!t.force_parts && t.force_fin == nullptr)) return 0;
  return ((nblk + 1 + W - 1) / W + 7) / 8 * 8;
}

namespace {
constexpr int kMaxDev = 64;

int device_cus(int dev) {
  static int cache[kMaxDev] = {0};
  if (dev < 0 || dev >= kMaxDev) dev = 0;
  if (cache[dev] == 0) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0)
      cus = 256;
    cache[dev] = cus;
  }
  return cache[dev];
}

int current_device() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDev) dev = 0;
  return dev;
}

// Workgroups of a kernel that are resident on the whole device at once
// (occupancy query, cached per device and kernel).
template <typename F>
int resident_blocks(F kernel, int threads, int* cache) {
  const int dev = current_device();
  if (cache[dev] == 0) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess ||
        per_cu <= 0)
      per_cu = 1;
    cache[dev] = per_cu * device_cus(dev);
  }
  return cache[dev];
}

int launch_error(std::string& err, const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    err = std::string(what) + ": " + hipGetErrorString(e);
    return -3;
  }
  return 0;
}

// Grid of the single-mesh stage kernel: persistent (at most the resident
// workgroups) or one tile per wave; a multiple of 8 either way.
int64_t stage_grid(int64_t ntiles, int waves, int resident, int mode) {
  const int64_t want = (ntiles + waves - 1) / waves;
  int64_t grid;
  if (mode == 1) {
    grid = (want + 7) / 8 * 8;
  } else if (mode >= 2) {
    // `mode` tiles per wave (at most the resident workgroups): every wave
    // does the same number of tiles, none waits on a partly filled last round
    const int64_t g = (ntiles + (int64_t)waves * mode - 1) / ((int64_t)waves * mode);
    grid = g < resident ? g : resident;
    grid = grid >= 8 ? (grid + 7) / 8 * 8 : 8;
    if (grid > resident) grid = resident / 8 * 8;
  } else {
    // a mesh that does not fill the chip takes one tile per wave: rounded
    // down, a few waves would take two and the launch twice the time (512
    // elements at p = 2 in seven-element tiles: 11.1 instead of 7 us)
    grid = (want + 7) / 8 * 8 < resident ? (want + 7) / 8 * 8 : resident / 8 * 8;
  }
  return grid < 8 ? 8 : grid;
}

}  // namespace

}  // namespace dgmi
