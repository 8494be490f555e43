// The stage from face traces for batches: many meshes in one launch per stage
// (all orders, or one order group), and the traces of their states at the
// start of a step.  A wave takes the tiles of one instance after the other,
// each run of them as trace_tiles does on a single mesh: the next tile's loads
// in flight during this one's work.
#include <hip/hip_runtime.h>

#include "trace_device.h"

namespace dgmi {

// The tiles of this workgroup's waves in group g: f(item, first tile, end tile
// of the item's own numbering, stride) for each instance they touch.
template <int W, typename F>
__device__ __forceinline__ void for_items(const BatchItem* __restrict__ items, const BatchGroup& g, F f) {
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int local = blockIdx.x - g.block_begin;
  const int xcd = local & 7;
  const int te = (int)(g.ntiles * (xcd + 1) / 8), stride = (g.nblocks >> 3) * W;
  int tile = (int)(g.ntiles * xcd / 8) + (local >> 3) * W + wid, i = g.first_item;
  while (tile < te) {
    while (tile >= items[i].tile_end) ++i;  // tiles only increase
    const int begin = (int)items[i].tile_begin;
    const int end = (int)items[i].tile_end < te ? (int)items[i].tile_end : te;
    f(i, tile - begin, end - begin, stride);
    tile += (end - tile + stride - 1) / stride * stride;
  }
}

template <int N, typename T, bool PERT, int W, bool LARGE>
__device__ __forceinline__ void batch_trace_group(const BatchItem* __restrict__ items,
                                                  const BatchStep* __restrict__ steps, int par,
                                                  const BatchGroup& g, int stage, double a, double b,
                                                  unsigned char* smem) {
  typedef typename Vec4<T>::type V4;
  using O = Order<N, T>;
  using P = TraceOrder<N, T, LARGE>;
  T* sFrag = (T*)smem;
  T* sWave = sFrag + O::FRAG_SZ;
  trace_lds_init<N, T, W, O::FRAG_SZ, LARGE, TraceOrder<N, T, LARGE>::WAVE_SZ>(frag_table<T>(items[g.first_item].t), sFrag, sWave);
  T* area = sWave + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * P::WAVE_SZ;
  for_items<W>(items, g, [&](int i, int tile0, int tile_end, int stride) {
    const BatchItem& it = items[i];
    KernelPhysics ph = it.ph;
    ph.vw[0] = steps[i].vw[0];
    ph.vw[1] = steps[i].vw[1];
    const int src = (par + stage) & 1;
    trace_tiles<N, T, PERT, LARGE, false>(it.t, ph, it.buf[src], it.buf[src ^ 1], it.K1, a, b, steps[i].dt,
                                   (const V4*)it.tr[src], (V4*)it.tr[src ^ 1], sFrag, area, tile0, tile_end, stride, [] {});
  });
}

template <typename T, int W, bool LARGE>
struct BatchTraceLds {
  template <int N>
  static constexpr size_t of() {
    return (Order<N, T>::FRAG_SZ + W * TraceOrder<N, T, LARGE>::WAVE_SZ) * sizeof(T);
  }
  static constexpr size_t mx(size_t x, size_t y) { return x > y ? x : y; }
  static constexpr size_t bytes = mx(mx(mx(of<1>(), of<2>()), mx(of<3>(), of<4>())), mx(of<5>(), of<6>()));
};

// All order groups in one launch: registers and LDS for the largest order.
template <typename T, bool PERT, int W, bool LARGE>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(2))) void
batch_trace_stage_kernel(const BatchItem* __restrict__ items, const BatchStep* __restrict__ steps,
                         const int* __restrict__ parity, BatchGroups G, int stage, double a, double b) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[BatchTraceLds<T, W, LARGE>::bytes];
  // the group of this workgroup, selected without dynamic indexing of the
  // by-value argument (which would place a copy of it in scratch memory)
  BatchGroup g = G.g[0];
#pragma unroll
  for (int k = 1; k < kMaxOrder; ++k)
    if (k < G.ng && (int)blockIdx.x >= G.g[k].block_begin) g = G.g[k];
  const int par = parity[0];
  switch (g.p) {
    case 1: batch_trace_group<1, T, PERT, W, LARGE>(items, steps, par, g, stage, a, b, smem); break;
    case 2: batch_trace_group<2, T, PERT, W, LARGE>(items, steps, par, g, stage, a, b, smem); break;
    case 3: batch_trace_group<3, T, PERT, W, LARGE>(items, steps, par, g, stage, a, b, smem); break;
    case 4: batch_trace_group<4, T, PERT, W, LARGE>(items, steps, par, g, stage, a, b, smem); break;
    case 5: batch_trace_group<5, T, PERT, W, LARGE>(items, steps, par, g, stage, a, b, smem); break;
    case 6: batch_trace_group<6, T, PERT, W, LARGE>(items, steps, par, g, stage, a, b, smem); break;
    default: break;
  }
}

// One order group per launch, sized for its own order.
template <int N, typename T, bool PERT, int W, bool LARGE>
__global__ __launch_bounds__(64 * W)
__attribute__((amdgpu_waves_per_eu(TraceOrder<N, T, LARGE>::MIN_WAVES_EU))) void
batch_trace_order_kernel(const BatchItem* __restrict__ items, const BatchStep* __restrict__ steps,
                         const int* __restrict__ parity, BatchGroup g, int stage, double a, double b) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[BatchTraceLds<T, W, LARGE>::template of<N>()];
  batch_trace_group<N, T, PERT, W, LARGE>(items, steps, parity[0], g, stage, a, b, smem);
}

// The traces of every instance of an order group (the first step on its states).
template <int N, typename T, bool PERT, bool LARGE>
__global__ __launch_bounds__(256) void batch_face_trace_kernel(const BatchItem* __restrict__ items,
                                                               const BatchStep* __restrict__ steps,
                                                               const int* __restrict__ parity, BatchGroup g) {
  constexpr int W = 4;
  using O = Order<N, T>;
  using P = TraceOrder<N, T, LARGE>;
  __shared__ __attribute__((aligned(16))) T sFrag[2 * O::FD];
  __shared__ __attribute__((aligned(16))) T sWave[W * P::WAVE_SZ];
  trace_lds_init<N, T, W, 2 * O::FD, LARGE, TraceOrder<N, T, LARGE>::WAVE_SZ>(frag_table<T>(items[g.first_item].t), sFrag, sWave);
  T* area = sWave + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * P::WAVE_SZ;
  const int par = parity[0];
  for_items<W>(items, g, [&](int i, int tile0, int tile_end, int stride) {
    const BatchItem& it = items[i];
    KernelPhysics ph = it.ph;
    ph.vw[0] = steps[i].vw[0];
    ph.vw[1] = steps[i].vw[1];
    for (int tile = tile0; tile < tile_end; tile += stride)
      trace_tile<N, T, PERT, LARGE>(it.t, ph, it.buf[par], (typename Vec4<T>::type*)it.tr[par], sFrag, area, tile);
  });
}

// The wall faces' traces of every instance for the step's wall velocities
// (workgroup y: instance y; one wave each): 6 us, where all traces anew take 165
// of the 1,900 us of a 16-cylinder step.
template <typename T, bool PERT>
__global__ __launch_bounds__(64) void batch_wall_trace_kernel(const BatchItem* __restrict__ items,
                                                              const BatchStep* __restrict__ steps,
                                                              const int* __restrict__ parity) {
  __shared__ T norms[64];
  const BatchItem& it = items[blockIdx.y];
  if ((int)blockIdx.x * (64 / (it.p + 1)) >= it.t.nwall) return;
  KernelPhysics ph = it.ph;
  ph.vw[0] = steps[blockIdx.y].vw[0];
  ph.vw[1] = steps[blockIdx.y].vw[1];
  const int par = parity[0];
  typename Vec4<T>::type* tr = (typename Vec4<T>::type*)it.tr[par];
  switch (it.p) {
    case 1: wall_traces<1, T, PERT>(it.t, ph, it.buf[par], tr, blockIdx.x, norms); break;
    case 2: wall_traces<2, T, PERT>(it.t, ph, it.buf[par], tr, blockIdx.x, norms); break;
    case 3: wall_traces<3, T, PERT>(it.t, ph, it.buf[par], tr, blockIdx.x, norms); break;
    case 4: wall_traces<4, T, PERT>(it.t, ph, it.buf[par], tr, blockIdx.x, norms); break;
    case 5: wall_traces<5, T, PERT>(it.t, ph, it.buf[par], tr, blockIdx.x, norms); break;
    case 6: wall_traces<6, T, PERT>(it.t, ph, it.buf[par], tr, blockIdx.x, norms); break;
    default: break;
  }
}

namespace {
// Calls f(T value, bool_constant<PERT>) for a form with traces.
template <bool B>
struct Flag {
  static constexpr bool value = B;
};
template <typename F>
int with_form(int form, std::string& err, F f) {
  switch (form) {
    case 0: return f(double(), Flag<false>());
    case 1: return f(double(), Flag<true>());
    case 2: return f(float(), Flag<true>());
    default: err = "face traces are not built for this form"; return -5;
  }
}
template <int N>
struct OrderTag {
  static constexpr int value = N;
};
template <typename F>
int with_order(int N, std::string& err, F f) {
  switch (N) {
    case 1: return f(OrderTag<1>());
    case 2: return f(OrderTag<2>());
    case 3: return f(OrderTag<3>());
    case 4: return f(OrderTag<4>());
    case 5: return f(OrderTag<5>());
    case 6: return f(OrderTag<6>());
    default: err = "polynomial order not built"; return -5;
  }
}
template <typename F>
int with_shape(int waves, bool large, std::string& err, F f) {
  if (waves == 2) return large ? f(OrderTag<2>(), Flag<true>()) : f(OrderTag<2>(), Flag<false>());
  if (waves == 4) return large ? f(OrderTag<4>(), Flag<true>()) : f(OrderTag<4>(), Flag<false>());
  err = "waves per workgroup must be 2 or 4";
  return -1;
}

template <int N, typename T, bool PERT, int W, bool LARGE>
int resident_order() {
  static int cache[kMaxDev] = {0};
  return resident_blocks(batch_trace_order_kernel<N, T, PERT, W, LARGE>, 64 * W, cache);
}
template <typename T, bool PERT, int W, bool LARGE>
int resident_all() {
  static int cache[kMaxDev] = {0};
  return resident_blocks(batch_trace_stage_kernel<T, PERT, W, LARGE>, 64 * W, cache);
}
template <int N, typename T, bool PERT, bool LARGE>
int resident_traces() {
  static int cache[kMaxDev] = {0};
  return resident_blocks(batch_face_trace_kernel<N, T, PERT, LARGE>, 256, cache);
}
}  // namespace

bool beyond_cache(int64_t bytes) { return bytes > kLastLevelCache; }
int64_t trace_stage_bytes(int N, int form, int64_t K) { return stage_bytes(N, form == 2 ? 4 : 8, K); }

int batch_trace_resident_blocks(int N, int form, int waves, bool large) {
  std::string err;
  return with_form(form, err, [&](auto x, auto pert) {
    typedef decltype(x) T;
    return with_shape(waves, large, err, [&](auto w, auto lg) {
      if (N == 0) return resident_all<T, decltype(pert)::value, decltype(w)::value, decltype(lg)::value>();
      return with_order(N, err, [&](auto n) {
        return resident_order<decltype(n)::value, T, decltype(pert)::value, decltype(w)::value, decltype(lg)::value>();
      });
    });
  });
}

int launch_batch_trace_stage(int form, int waves, bool large, const BatchItem* items, const BatchStep* steps,
                             const int* parity, const BatchGroups& G, int blocks, int stage, double a, double b,
                             void* stream, std::string& err) {
  return with_form(form, err, [&](auto x, auto pert) {
    typedef decltype(x) T;
    return with_shape(waves, large, err, [&](auto w, auto lg) {
      constexpr int W = decltype(w)::value;
      hipLaunchKernelGGL((batch_trace_stage_kernel<T, decltype(pert)::value, W, decltype(lg)::value>),
                         dim3((unsigned)blocks), dim3(64 * W), 0, (hipStream_t)stream, items, steps, parity, G,
                         stage, a, b);
      return launch_error(err, "batched trace stage launch");
    });
  });
}

int launch_batch_trace_order_stage(int N, int form, int waves, bool large, const BatchItem* items,
                                   const BatchStep* steps, const int* parity, const BatchGroup& g, int blocks,
                                   int stage, double a, double b, void* stream, std::string& err) {
  return with_form(form, err, [&](auto x, auto pert) {
    typedef decltype(x) T;
    return with_shape(waves, large, err, [&](auto w, auto lg) {
      return with_order(N, err, [&](auto n) {
        constexpr int W = decltype(w)::value;
        hipLaunchKernelGGL(
            (batch_trace_order_kernel<decltype(n)::value, T, decltype(pert)::value, W, decltype(lg)::value>),
            dim3((unsigned)blocks), dim3(64 * W), 0, (hipStream_t)stream, items, steps, parity, g, stage, a, b);
        return launch_error(err, "batched trace stage launch");
      });
    });
  });
}

int launch_batch_wall_traces(int form, const BatchItem* items, const BatchStep* steps, const int* parity,
                             int n_items, int max_blocks, void* stream, std::string& err) {
  return with_form(form, err, [&](auto x, auto pert) {
    hipLaunchKernelGGL((batch_wall_trace_kernel<decltype(x), decltype(pert)::value>),
                       dim3((unsigned)max_blocks, (unsigned)n_items), dim3(64), 0, (hipStream_t)stream, items, steps,
                       parity);
    return launch_error(err, "wall trace launch");
  });
}

int launch_batch_face_traces(int form, bool large, const BatchItem* items, const BatchStep* steps,
                             const int* parity, BatchGroup g, void* stream, std::string& err) {
  return with_form(form, err, [&](auto x, auto pert) {
    typedef decltype(x) T;
    return with_shape(4, large, err, [&](auto, auto lg) {
      return with_order(g.p, err, [&](auto n) {
        constexpr int N = decltype(n)::value;
        constexpr bool PERT = decltype(pert)::value, LARGE = decltype(lg)::value;
        g.block_begin = 0;
        g.nblocks = (int)stage_grid(g.ntiles, 4, resident_traces<N, T, PERT, LARGE>(), 0);
        hipLaunchKernelGGL((batch_face_trace_kernel<N, T, PERT, LARGE>), dim3((unsigned)g.nblocks), dim3(256), 0,
                           (hipStream_t)stream, items, steps, parity, g);
        return launch_error(err, "batched face trace launch");
      });
    });
  });
}

}  // namespace dgmi
