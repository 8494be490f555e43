// Launch-shape selection of the stage kernels: set/get, and an autotuner that
// times every shape on the context's own mesh, with a JSON-lines cache.  A
// context has two shapes, of the stage from the neighbours' states (dg_rhs,
// dg_rk_stage, single steps on small meshes) and of the one from face traces
// (steps): different kernels with different registers and LDS.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>

#include "dg_ctx.h"

namespace {

// One line: the steps' kernel ("traces" or "states"), its shape and time, and the
// shape of the stage from the states.  Lines of another form are passed over.
struct CacheEntry {
  char arch[96], kernel[16];
  int p, precision, curved;
  long long K;
  int waves, grid, stage_waves, stage_grid;
  double us;
};

bool valid_shape(int waves, int grid) {
  return (waves == 0 || waves == 2 || waves == 4) && (grid >= 0 && grid <= 3);
}

bool parse_line(const char* line, CacheEntry& e) {
  return std::sscanf(line,
                     "{\"arch\": \"%95[^\"]\", \"p\": %d, \"precision\": %d, \"K\": %lld, "
                     "\"kernel\": \"%15[^\"]\", \"curved\": %d, \"waves\": %d, \"grid\": %d, "
                     "\"stage_waves\": %d, \"stage_grid\": %d, \"us\": %lf}",
                     e.arch, &e.p, &e.precision, &e.K, e.kernel, &e.curved, &e.waves, &e.grid,
                     &e.stage_waves, &e.stage_grid, &e.us) == 11 &&
         valid_shape(e.waves, e.grid) && valid_shape(e.stage_waves, e.stage_grid);
}

// Closest cached entry (in K, within a factor 2) for this architecture, order and
// precision, the same kernel of the steps, with or without curved elements.
bool cache_lookup(const char* path, const char* arch, int p, int precision, long long K,
                  const char* kernel, int curved, CacheEntry& best) {
  FILE* f = std::fopen(path, "r");
  if (!f) return false;
  char line[512];
  bool found = false;
  double bestd = 0.0;
  while (std::fgets(line, sizeof line, f)) {
    CacheEntry e;
    if (!parse_line(line, e)) continue;
    if (std::strcmp(e.arch, arch) != 0 || e.p != p || e.precision != precision) continue;
    if (std::strcmp(e.kernel, kernel) != 0 || (e.curved != 0) != (curved != 0)) continue;
    if (e.K > 2 * K || 2 * e.K < K) continue;
    const double d = e.K > K ? (double)e.K / K : (double)K / e.K;
    if (!found || d < bestd) {
      best = e;
      bestd = d;
      found = true;
    }
  }
  std::fclose(f);
  return found;
}

// Time every launch shape of the stages' kernel (stages.tr: from traces or from
// the states) on U, a later RK stage (A_2 != 0), as four of the five are: reads U
// and K1, writes scratch and K1 (and traces, where the steps do).
int time_shapes(dg_ctx* c, dgmi::Stages stages, const double* U, double* K1, int sweeps, int warm, int reps,
                hipStream_t s, hipEvent_t e0, hipEvent_t e1, dgmi::StageTuning& pick, double& best) {
  const dgmi::DeviceTables t = dgmi::ctx_tables(c);
  const double vw0[2] = {0.0, 0.0};
  const dgmi::KernelPhysics ph = dgmi::ctx_phys(c, vw0);
  std::string err;
  if (stages.begin(t, ph, U, s, err) != 0) return dgmi::ctx_fail(c, DG_EHIP, err);
  auto go = [&]() {
    stages.in = 0;
    return stages.run(t, ph, U, c->d_scratch, K1, 1, 1e-7, false, s, err);
  };
  best = 1e300;
  // each shape's best time over the sweeps is kept: the candidates are often within
  // a few per cent, and one sweep's clock drift or noise could pick the slower one
  constexpr int kShapes = 8;
  double shape_us[kShapes];
  for (double& x : shape_us) x = 1e300;
  for (int sweep = 0; sweep < sweeps; ++sweep)
    for (int w : {2, 4})
      for (int grid = 0; grid < 4; ++grid) {
        stages.tune.waves = w;
        stages.tune.grid = grid;
        for (int r = 0; r < warm; ++r)
          if (go() != 0) return dgmi::ctx_fail(c, DG_EHIP, err);
        (void)hipEventRecord(e0, s);
        for (int r = 0; r < reps; ++r)
          if (go() != 0) return dgmi::ctx_fail(c, DG_EHIP, err);
        (void)hipEventRecord(e1, s);
        const hipError_t e = hipEventSynchronize(e1);
        if (e != hipSuccess) return dgmi::ctx_hip_fail(c, e, "hipEventSynchronize");
        float ms = 0.f;
        (void)hipEventElapsedTime(&ms, e0, e1);
        const double us = 1e3 * ms / reps;
        double& sb = shape_us[(w == 4 ? 4 : 0) + grid];
        if (us < sb) sb = us;
        if (sweep == sweeps - 1 && sb < best) {
          best = sb;
          pick = stages.tune;
        }
      }
  return DG_OK;
}

}  // namespace

extern "C" {

int dg_set_tuning(dg_ctx* c, int waves, int grid) {
  if (!c) return DG_EINVAL;
  if (!valid_shape(waves, grid)) return dgmi::ctx_fail(c, DG_EINVAL, "waves 0/2/4, grid 0..3");
  // the shape that dg_get_tuning reports changes nothing, whichever shapes (the
  // default, the autotuner's) the two kernels have
  int now_waves = 0, now_grid = 0;
  if (dg_get_tuning(c, &now_waves, &now_grid) == DG_OK && waves == now_waves && grid == now_grid) return DG_OK;
  c->tune.waves = waves;
  c->tune.grid = grid;
  c->tune_traces = c->tune;
  return DG_OK;
}

int dg_get_tuning(const dg_ctx* c, int* waves, int* grid) {
  if (!c || !waves || !grid) return DG_EINVAL;
  const bool traces = dgmi::steps_from_traces(c);
  const dgmi::StageTuning& t = traces ? c->tune_traces : c->tune;
  *waves = t.waves ? t.waves
                   : (traces ? dgmi::default_trace_waves(c->N, dgmi::ctx_form(c), c->K)
                             : (c->overint ? 2 : dgmi::default_waves(c->N, c->precision)));
  *grid = t.grid;
  return DG_OK;
}

int dg_autotune(dg_ctx* c, const double* U, int reps, const char* cache_path, void* stream,
                double* best_us) {
  if (!c) return DG_EINVAL;
  if (!c->dev_ready) return dgmi::ctx_fail(c, DG_ESTATE, "dg_setup has not completed");
  if (!U || reps < 1) return dgmi::ctx_fail(c, DG_EINVAL, "U is NULL or reps < 1");
  hipDeviceProp_t prop;
  hipError_t e = hipGetDeviceProperties(&prop, c->device);
  if (e != hipSuccess) return dgmi::ctx_hip_fail(c, e, "hipGetDeviceProperties");
  char arch[96];
  std::snprintf(arch, sizeof arch, "%s", prop.gcnArchName);
  for (char* q = arch; *q; ++q)
    if (*q == '"' || *q == '\\') *q = '_';
  dgmi::ctx_steps_memory(c, 2, stream);
  const dgmi::Stages stages = dgmi::ctx_stages(c, 2);
  const char* kernel = stages.tr[0] ? "traces" : "states";
  const int curved = c->mesh.celem.empty() ? 0 : 1;
  if (cache_path) {
    CacheEntry hit;
    if (cache_lookup(cache_path, arch, c->N, dgmi::ctx_form(c), (long long)c->K, kernel, curved, hit)) {
      c->tune.waves = hit.stage_waves;
      c->tune.grid = hit.stage_grid;
      c->tune_traces.waves = hit.waves;
      c->tune_traces.grid = hit.grid;
      if (best_us) *best_us = 0.0;
      return DG_OK;
    }
  }
  hipStream_t s = (hipStream_t)stream;
  const size_t bytes = (size_t)c->K * 4 * c->ref.Np * sizeof(double);
  double* K1 = nullptr;
  e = hipMalloc((void**)&K1, bytes);
  if (e != hipSuccess) return dgmi::ctx_hip_fail(c, e, "hipMalloc");
  hipEvent_t e0 = nullptr, e1 = nullptr;
  e = hipEventCreate(&e0);
  if (e == hipSuccess) e = hipEventCreate(&e1);
  int rc = DG_OK;
  double best = 1e300;
  dgmi::StageTuning stage_pick, pick;
  if (e != hipSuccess) rc = dgmi::ctx_hip_fail(c, e, "hipEventCreate");
  if (rc == DG_OK && (e = hipMemsetAsync(K1, 0, bytes, s)) != hipSuccess)
    rc = dgmi::ctx_hip_fail(c, e, "hipMemsetAsync");
  // the kernel of the steps in two sweeps; where that is the one from traces, the
  // stage from the states beside it in a quick one, a fifteenth of the time (in full,
  // tuning 20,480 elements at p = 4 in FP64 would take twice its 12 ms)
  if (rc == DG_OK) rc = time_shapes(c, stages, U, K1, 2, 3, reps, s, e0, e1, pick, best);
  stage_pick = pick;
  double stage_best = best;
  if (rc == DG_OK && stages.tr[0])
    rc = time_shapes(c, dgmi::Stages(c, nullptr, nullptr), U, K1, 1, 1, reps > 16 ? reps / 8 : 2, s, e0, e1, stage_pick,
                     stage_best);
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  (void)hipFree(K1);
  if (rc != DG_OK) return rc;
  c->tune = stage_pick;
  c->tune_traces = pick;
  if (best_us) *best_us = best;
  if (cache_path) {
    FILE* f = std::fopen(cache_path, "a");
    if (!f) return dgmi::ctx_fail(c, DG_EINVAL, std::string("cannot append to ") + cache_path);
    std::fprintf(f,
                 "{\"arch\": \"%s\", \"p\": %d, \"precision\": %d, \"K\": %lld, \"kernel\": \"%s\", "
                 "\"curved\": %d, \"waves\": %d, \"grid\": %d, \"stage_waves\": %d, \"stage_grid\": %d, "
                 "\"us\": %.3f}\n",
                 arch, c->N, dgmi::ctx_form(c), (long long)c->K, kernel, curved, pick.waves, pick.grid,
                 stage_pick.waves, stage_pick.grid, best);
    std::fclose(f);
  }
  return DG_OK;
}

}  // extern "C"
