// The context behind the opaque dg_ctx handle, and helpers shared by the
// C-ABI sources (dgmi_abi.cpp, batch.cpp, tune.cpp).
#pragma once

#include <hip/hip_runtime.h>

#include <string>
#include <vector>

#include "../../include/dgmi.h"
#include "dg_internal.h"

namespace dgmi {
// Carpenter & Kennedy (1994) five-stage, fourth-order 2N-storage coefficients
// (NASA TM-109112): K1 <- A_i K1 + dt R(K0), K0 <- K0 + B_i K1 (Alg. 1).
constexpr double kRkA[5] = {0.0, -567301805773.0 / 1357537059087.0,
                            -2404267990393.0 / 2016746695238.0,
                            -3550918686646.0 / 2091501179385.0,
                            -1275806237668.0 / 842570457699.0};
constexpr double kRkB[5] = {1432997174477.0 / 9575080441755.0, 5161836677717.0 / 13612068292357.0,
                            1720146321549.0 / 2090206949498.0, 3134564353537.0 / 4481467310338.0,
                            2277821191437.0 / 14882151754819.0};
}  // namespace dgmi

struct dg_ctx {
  int N = 0;
  int precision = 0;
  dgmi::StageTuning tune;         // of the stage from the neighbours' states
  dgmi::StageTuning tune_traces;  // of the stage from face traces
  dgmi::Physics phys;
  bool have_phys = false;
  std::vector<double> VX, VY;
  std::vector<int32_t> EToV;
  std::vector<int8_t> tag;
  double period[2] = {0.0, 0.0};
  int64_t Nv = 0, K = 0;
  bool have_mesh = false;
  dgmi::RefOps ref;
  dgmi::MeshTables mesh;
  bool host_ready = false;
  int device = -1;
  double* d_geo = nullptr;
  int32_t* d_conn = nullptr;
  double* d_ops = nullptr;
  double* d_frag = nullptr;
  double* d_oi = nullptr;         // over-integration fragments and tables
  int64_t oi_len = 0;
  dgmi::OIOps oi;
  bool overint = false;
  float* d_frag32 = nullptr;
  uint16_t* d_frag16 = nullptr;
  int32_t* d_wall = nullptr;
  double* d_wall_xy = nullptr;
  double* d_scratch = nullptr;
  double* d_scratch2 = nullptr;   // a second scratch state (null: an odd number of stages ends with a copy)
  void* d_trace[2] = {nullptr, nullptr};  // face traces of a stage's input and output (null: none)
  size_t trace_size = 0;                  // bytes of each
  bool no_trace_memory = false, no_scratch2_memory = false;  // found too little memory for them
  std::vector<void*> retired;             // earlier, smaller trace arrays
  double* h_force = nullptr;        // pinned: partials of the force the host sums
  double* d_force_part = nullptr;
  unsigned* d_force_ticket = nullptr;
  double* d_cfl = nullptr;          // CFL work: 3K face maxima, 3K element maxima
  double* h_cfl = nullptr;          // pinned: the CFL bound's maxima by workgroup
  double* noalloc_scratch = nullptr;  // this device's static scratch array (not owned)
  // isoparametric elements given by dg_set_curved_elements, and their tables
  std::vector<int32_t> curved_elems;
  std::vector<double> curved_xy;
  int32_t* d_cslot = nullptr;
  int32_t* d_celem = nullptr;
  double* d_cnode = nullptr;
  double* d_cface = nullptr;
  double* d_cP = nullptr;
  int force_blocks = 0;
  bool dev_ready = false;
  std::string err;
};

namespace dgmi {
int ctx_fail(dg_ctx* c, int code, const std::string& msg);
int ctx_hip_fail(dg_ctx* c, hipError_t e, const char* what);
DeviceTables ctx_tables(const dg_ctx* c);
// the form launch_stage runs for this context (its precision mode, or the
// over-integrated FP64 stage)
inline int ctx_form(const dg_ctx* c) { return c->overint ? kFormOverint : c->precision; }
KernelPhysics ctx_phys(const dg_ctx* c, const double vw[2]);
// Whether memory that a call can do without may be taken: at most half of what
// is free on the current device, the rest for what a program cannot.
inline bool leaves_half(size_t bytes) {
  size_t room = 0, total = 0;
  return hipMemGetInfo(&room, &total) == hipSuccess && bytes <= room / 2;
}
// The stages of one multi-step call: from face traces where the call has
// buffers for them (tr), else from the neighbours' states.  begin() takes the
// call's first state; the last stage of the call leaves no traces.
struct Stages {
  int N, form;
  StageTuning tune;
  void* tr[2];
  int in = 0;
  Stages(const dg_ctx* c, void* tr0, void* tr1) : N(c->N), form(ctx_form(c)), tune(tr0 ? c->tune_traces : c->tune), tr{tr0, tr1} {}
  int begin(const DeviceTables& t, const KernelPhysics& ph, const double* U, void* stream, std::string& err) {
    return tr[0] ? launch_face_traces(N, form, t, ph, U, tr[in], stream, err) : 0;
  }
  int run(const DeviceTables& t, const KernelPhysics& ph, const double* Uin, double* Uout, double* K1, int i,
          double dt, bool last, void* stream, std::string& err) {
    if (!tr[0]) return launch_stage(N, form, tune, t, ph, Uin, Uout, K1, kRkA[i], kRkB[i], dt, 0, stream, err);
    const int rc = launch_trace_stage(N, form, tune, t, ph, Uin, Uout, K1, kRkA[i], kRkB[i], dt, tr[in],
                                      last ? nullptr : tr[in ^ 1], stream, err);
    in ^= 1;
    return rc;
  }
};
// The state buffers of one call's stages: U and a scratch state in turn.  An odd
// number of stages goes U, S, S2, U at its start where there is a second scratch
// state, and so ends in U; else it ends in the scratch state (in_scratch).
struct StateBuffers {
  double *U, *S, *S2;
  bool odd;
  StateBuffers(double* u, double* s, double* s2, int64_t stages) : U(u), S(s), S2(stages >= 3 ? s2 : nullptr), odd(stages & 1) {}
  // the state before stage i, which is the output of stage i - 1
  double* at(int64_t i) const {
    if (odd && S2) return i < 3 ? (i == 0 ? U : (i == 1 ? S : S2)) : ((i & 1) ? U : S);
    return (i & 1) ? S : U;
  }
  bool in_scratch() const { return odd && !S2; }
};
// The memory that multi-step calls use and can do without -- face traces and a
// second scratch state -- is taken by the first call that has a use for it (a
// context that only serves single stages, or a batch, holds none), unless that
// call is being captured: it then runs as where the memory is short, from the
// neighbours' states and with a copy at the end of an odd number of steps.
void ctx_steps_memory(dg_ctx* c, int nsteps, void* stream);
// The largest state that gets a second scratch state: beyond it the copy that
// this saves is 3 % of a step's five stages (20,480 elements at p = 4: 3 of 90
// us; the smaller the mesh, the more: 5,120 at p = 3: 3 us and a launch of 62).
constexpr size_t kSecondScratch = (size_t)64 << 20;
// Face traces serve every form but bfloat16 operators, and meshes with curved
// elements where the stage's arrays fit the last-level cache (beyond it the
// stages run from the neighbours' states).  A side takes the other's normal flux
// with the sign changed, so they do not serve a mesh with a periodic seam whose
// sides have other normals (vertices that are not exact translates).
inline size_t ctx_trace_bytes(const dg_ctx* c) {
  const int form = ctx_form(c);
  if (!c->mesh.opposed) return 0;
  if (!c->mesh.celem.empty() && (form == kFormOverint || beyond_cache(trace_stage_bytes(c->N, form, c->K)))) return 0;
  return trace_bytes(c->N, form, c->K);
}
// Whether nsteps steps on K elements of one mesh run from traces:
// the launch that makes the first ones costs 6 us on a small mesh, which the
// five stages of a single step win back from about 16,000 elements on (one
// step at p = 4 FP32: 8,192 elements 59.3 against 56.2 us, 20,480 93.9 against
// 95.9), in FP64 at p >= 5 always (512 elements 106.8 against 114.2 us).
// At p = 1 in FP64 the eight-element tile is the longer one where the mesh
// does not fill the chip (2,560 elements 8.2 against 7.6 us a stage, 8,192 8.6
// against 9.7).
inline bool traces_pay(int N, int form, int64_t K, int nsteps) {
  if (form == kFormOverint) return true;
  if (N == 1 && form != 2 && K < 8192) return false;
  return nsteps > 1 || K >= 16384 || (form != 2 && N >= 5);
}
inline Stages ctx_stages(const dg_ctx* c, int nsteps) {
  const size_t need = ctx_trace_bytes(c);
  const bool use = need > 0 && need <= c->trace_size && traces_pay(c->N, ctx_form(c), c->K, nsteps);
  return Stages(c, use ? c->d_trace[0] : nullptr, use ? c->d_trace[1] : nullptr);
}
// Whether several steps of this context run from traces (or will, once the first
// of them has taken the memory).
inline bool steps_from_traces(const dg_ctx* c) {
  return ctx_trace_bytes(c) > 0 && !c->no_trace_memory && traces_pay(c->N, ctx_form(c), c->K, 2);
}
// noalloc.hip: device address of the static scratch array on the current
// device (looked up once per device); its size in bytes
int noalloc_scratch_address(double** out, std::string& err);
size_t noalloc_scratch_bytes();
}  // namespace dgmi
