// The stage from face traces on a single mesh: kernels and launches.
#include <hip/hip_runtime.h>

#include "curved_device.h"
#include "trace_device.h"

namespace dgmi {

// Single mesh, tiles per XCD as in stage_kernel; the leading workgroups take
// the curved set (CURVED: one element per wave, with its traces), then the wall
// force of the input state and the sum of the previous partials.  20,320 straight
// elements and 160 of the set, p = 4 FP32: 21.4 us a stage from the neighbours'
// states, 19.7 from traces; the longest then is a curved wave's chain of dependent
// phases, with the straight tiles beside it.
template <int N, typename T, bool CURVED>
constexpr int wave_lds(int tile_size) {
  const int curved = (int)((curved_lds_doubles(N) + 1) * sizeof(double) / sizeof(T));
  return CURVED && curved > tile_size ? (curved + 3) / 4 * 4 : tile_size;
}
template <int N, typename T, bool PERT, int W, bool LARGE, bool CURVED>
__global__ __launch_bounds__(64 * W)
__attribute__((amdgpu_waves_per_eu(TraceOrder<N, T>::MIN_WAVES_EU))) void
trace_stage_kernel(DeviceTables t, KernelPhysics ph, const double* __restrict__ Uin,
                   double* __restrict__ Uout, double* __restrict__ K1, double a, double b, double dt,
                   const typename Vec4<T>::type* __restrict__ tr_in,
                   typename Vec4<T>::type* __restrict__ tr_out) {
  using P = TraceOrder<N, T, LARGE>;
  using O = Order<N, T>;
  __shared__ __attribute__((aligned(16))) T sFrag[O::FRAG_SZ];
  constexpr int WS = wave_lds<N, T, CURVED>(P::WAVE_SZ);
  __shared__ __attribute__((aligned(16))) T sWave[W * WS];
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ncw = CURVED ? curved_workgroups(t.ncurved, W) : 0;
  if constexpr (CURVED) {
    if ((int)blockIdx.x < ncw) {
      const int slot = (int)blockIdx.x * W + wid;
      if (slot < t.ncurved) {
        const uintptr_t at = ((uintptr_t)(sWave + wid * WS) + 7) & ~(uintptr_t)7;
        double* lds = (double*)at;
        curved_element<N>(t, ph, Uin, Uout, K1, a, b, dt, 0, slot, lds);
        wave_sync();
        // (the state leads the element's arrays; the next ones are free)
        if (tr_out != nullptr) element_traces<N, T, PERT>(t, ph, lds, t.celem[slot], tr_out, (T*)(lds + P::S));
      }
      return;
    }
  }
  const int nfw = force_workgroups(t, P::Nfp, W);
  if ((int)blockIdx.x < ncw + nfw) {
    const unsigned nblk = (unsigned)((t.nwall * P::Nfp + kForceThreads - 1) / kForceThreads);
    const unsigned wv = (blockIdx.x - ncw) * W + wid;
    if (t.force_parts && wv < nblk) force_wave<N, 8, false>(t, ph, Uin, nullptr, wv, nblk);
    if (t.force_fin != nullptr && wv == nblk) force_sum(t.force_part, t.force_fin, nblk);
    return;
  }
  const unsigned bx = blockIdx.x - ncw - nfw, gx = gridDim.x - ncw - nfw;
  const int64_t ntiles = (t.K + P::EPT - 1) / P::EPT;
  const int xcd = bx & 7;
  const int64_t tb = ntiles * xcd / 8, te = ntiles * (xcd + 1) / 8;
  const int64_t w0 = (int64_t)(bx >> 3) * W + wid;
  const int64_t wstride = (int64_t)(gx >> 3) * W;
  trace_tiles<N, T, PERT, LARGE, CURVED>(
      t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, sFrag, sWave + wid * WS, tb + w0, te, wstride,
      [&] { trace_lds_init<N, T, W, O::FRAG_SZ, LARGE, WS>(frag_table<T>(t), sFrag, sWave); });
}

template <int N, typename T, bool PERT, int W>
__global__ __launch_bounds__(64 * W) void face_trace_kernel(DeviceTables t, KernelPhysics ph,
                                                            const double* __restrict__ U,
                                                            typename Vec4<T>::type* __restrict__ tr) {
  using P = TraceOrder<N, T>;
  using O = Order<N, T>;
  __shared__ __attribute__((aligned(16))) T sFrag[2 * O::FD];
  __shared__ __attribute__((aligned(16))) T sWave[W * P::WAVE_SZ];
  trace_lds_init<N, T, W, 2 * O::FD, false, P::WAVE_SZ>(frag_table<T>(t), sFrag, sWave);
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t ntiles = (t.K + P::EPT - 1) / P::EPT;
  const int xcd = blockIdx.x & 7;
  const int64_t tb = ntiles * xcd / 8, te = ntiles * (xcd + 1) / 8;
  for (int64_t tile = tb + (int64_t)(blockIdx.x >> 3) * W + wid; tile < te; tile += (int64_t)(gridDim.x >> 3) * W)
    trace_tile<N, T, PERT, false>(t, ph, U, tr, sFrag, sWave + wid * P::WAVE_SZ, tile);
}

namespace {
template <int N, typename T, bool PERT, int W, bool LARGE, bool CURVED = false>
int launch_trace_stage_t(const StageTuning& tune, const DeviceTables& t, const KernelPhysics& ph,
                         const double* Uin, double* Uout, double* K1, double a, double b, double dt,
                         const void* tr_in, void* tr_out, hipStream_t s, std::string& err) {
  typedef typename Vec4<T>::type V4;
  static int cache[kMaxDev] = {0};
  const int resident = resident_blocks(trace_stage_kernel<N, T, PERT, W, LARGE, CURVED>, 64 * W, cache);
  constexpr int EPT = TraceOrder<N, T, LARGE>::EPT;
  // (the curved set keeps its resident slots beside a persistent grid)
  const int ncw = CURVED ? curved_workgroups(t.ncurved, W) : 0;
  const int straight_resident = resident - ncw >= 8 ? resident - ncw : 8;
  const int64_t grid =
      stage_grid((t.K + EPT - 1) / EPT, W, straight_resident, tune.grid) + ncw + force_workgroups(t, N + 1, W);
  hipLaunchKernelGGL((trace_stage_kernel<N, T, PERT, W, LARGE, CURVED>), dim3((unsigned)grid), dim3(64 * W), 0, s, t, ph, Uin,
                     Uout, K1, a, b, dt, (const V4*)tr_in, (V4*)tr_out);
  return launch_error(err, "trace stage kernel launch");
}

template <int N, typename T, bool PERT>
int launch_trace_stage_w(const StageTuning& tune, const DeviceTables& t, const KernelPhysics& ph,
                         const double* Uin, double* Uout, double* K1, double a, double b, double dt,
                         const void* tr_in, void* tr_out, hipStream_t s, std::string& err) {
  const int w = tune.waves ? tune.waves : TraceOrder<N, T>::WAVES;
  const bool stream = stage_bytes(N, sizeof(T), t.K) > kLastLevelCache;
  if (t.ncurved > 0 && (w == 2 || w == 4)) {
    if (stream) {
      err = "face traces are not built for curved elements beyond the last-level cache";
      return -5;
    }
    return w == 2 ? launch_trace_stage_t<N, T, PERT, 2, false, true>(tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in,
                                                                     tr_out, s, err)
                  : launch_trace_stage_t<N, T, PERT, 4, false, true>(tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in,
                                                                     tr_out, s, err);
  }
  if (w == 2 && stream)
    return launch_trace_stage_t<N, T, PERT, 2, true>(tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
  if (w == 2)
    return launch_trace_stage_t<N, T, PERT, 2, false>(tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
  if (w == 4 && stream)
    return launch_trace_stage_t<N, T, PERT, 4, true>(tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
  if (w == 4)
    return launch_trace_stage_t<N, T, PERT, 4, false>(tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
  err = "waves per workgroup must be 2 or 4";
  return -1;
}

template <int N, typename T, bool PERT>
int launch_face_traces_t(const DeviceTables& t, const KernelPhysics& ph, const double* U, void* tr, hipStream_t s,
                         std::string& err) {
  constexpr int W = 4, EPT = TraceOrder<N, T>::EPT;
  static int cache[kMaxDev] = {0};
  const int resident = resident_blocks(face_trace_kernel<N, T, PERT, W>, 64 * W, cache);
  const int64_t grid = stage_grid((t.K + EPT - 1) / EPT, W, resident, 0);
  hipLaunchKernelGGL((face_trace_kernel<N, T, PERT, W>), dim3((unsigned)grid), dim3(64 * W), 0, s, t, ph, U,
                     (typename Vec4<T>::type*)tr);
  return launch_error(err, "face trace kernel launch");
}

template <int N>
int launch_trace_stage_n(int form, const StageTuning& tune, const DeviceTables& t, const KernelPhysics& ph,
                         const double* Uin, double* Uout, double* K1, double a, double b, double dt,
                         const void* tr_in, void* tr_out, hipStream_t s, std::string& err) {
  switch (form) {
    case 0: return launch_trace_stage_w<N, double, false>(tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
    case 1: return launch_trace_stage_w<N, double, true>(tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
    case 2: return launch_trace_stage_w<N, float, true>(tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
    default: err = "face traces are not built for this form"; return -5;
  }
}

template <int N>
int launch_face_traces_n(int form, const DeviceTables& t, const KernelPhysics& ph, const double* U, void* tr,
                         hipStream_t s, std::string& err) {
  switch (form) {
    case 0: return launch_face_traces_t<N, double, false>(t, ph, U, tr, s, err);
    case 1: return launch_face_traces_t<N, double, true>(t, ph, U, tr, s, err);
    case 2: return launch_face_traces_t<N, float, true>(t, ph, U, tr, s, err);
    default: err = "face traces are not built for this form"; return -5;
  }
}
}  // namespace

size_t trace_bytes(int N, int form, int64_t K) {
  if (form == kFormOverint) return (size_t)K * 3 * oi_points(N) * 8 * sizeof(double);
  if (form < 0 || form > 2) return 0;
  return (size_t)K * 3 * (N + 1) * 4 * (form == 2 ? sizeof(float) : sizeof(double));
}

int default_trace_waves(int N, int form, int64_t K) {
  return form == kFormOverint ? default_oi_trace_waves(N, K) : TraceOrder<1, double>::WAVES;
}

int launch_trace_stage(int N, int form, const StageTuning& tune, const DeviceTables& t, const KernelPhysics& ph,
                       const double* Uin, double* Uout, double* K1, double a, double b, double dt,
                       const void* tr_in, void* tr_out, void* stream, std::string& err) {
  hipStream_t s = (hipStream_t)stream;
  if (form == kFormOverint)
    return launch_oi_trace_stage(N, tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, stream, err);
  switch (N) {
    case 1: return launch_trace_stage_n<1>(form, tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
    case 2: return launch_trace_stage_n<2>(form, tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
    case 3: return launch_trace_stage_n<3>(form, tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
    case 4: return launch_trace_stage_n<4>(form, tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
    case 5: return launch_trace_stage_n<5>(form, tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
    case 6: return launch_trace_stage_n<6>(form, tune, t, ph, Uin, Uout, K1, a, b, dt, tr_in, tr_out, s, err);
    default: err = "polynomial order not built"; return -5;
  }
}

int launch_face_traces(int N, int form, const DeviceTables& t, const KernelPhysics& ph, const double* U, void* tr,
                       void* stream, std::string& err) {
  hipStream_t s = (hipStream_t)stream;
  if (form == kFormOverint) return launch_oi_face_traces(N, t, ph, U, tr, stream, err);
  switch (N) {
    case 1: return launch_face_traces_n<1>(form, t, ph, U, tr, s, err);
    case 2: return launch_face_traces_n<2>(form, t, ph, U, tr, s, err);
    case 3: return launch_face_traces_n<3>(form, t, ph, U, tr, s, err);
    case 4: return launch_face_traces_n<4>(form, t, ph, U, tr, s, err);
    case 5: return launch_face_traces_n<5>(form, t, ph, U, tr, s, err);
    case 6: return launch_face_traces_n<6>(form, t, ph, U, tr, s, err);
    default: err = "polynomial order not built"; return -5;
  }
}

}  // namespace dgmi
