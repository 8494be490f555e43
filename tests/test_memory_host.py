"""Device memory of contexts and batches, counted on the CPU.

A child process loads a stand-in for the HIP runtime's memory, stream and launch
calls ahead of the library (device memory is host memory with a budget, kernels
do nothing), so that set-up, batch creation and steps run without a GPU and an
allocation past the budget fails as it would on one.
"""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2508_17917_amd", "libdgmi.so")
pytestmark = [pytest.mark.skipif(not os.path.exists(LIB), reason="libdgmi.so not built"),
              pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")]

SHIM = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
static std::map<void*, size_t> blocks;
static size_t used = 0, budget = (size_t)1 << 40;
static int capturing = 0;
extern "C" {
size_t shim_used() { return used; }
void shim_budget(size_t b) { budget = b; }
void shim_capturing(int c) { capturing = c; }
int hipMalloc(void** p, size_t n) {
  if (capturing) return 900;
  if (used + n > budget) return 2;
  *p = malloc(n ? n : 1);
  blocks[*p] = n;
  used += n;
  return 0;
}
int hipFree(void* p) {
  auto it = blocks.find(p);
  if (it == blocks.end()) return p ? 1 : 0;
  used -= it->second;
  blocks.erase(it);
  free(p);
  return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) { *p = malloc(n ? n : 1); return 0; }
int hipHostFree(void* p) { free(p); return 0; }
int hipMemGetInfo(size_t* f, size_t* t) { *f = budget > used ? budget - used : 0; *t = budget; return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { memcpy(d, s, n); return 0; }
int hipMemset(void* d, int v, size_t n) { memset(d, v, n); return 0; }
int hipMemsetAsync(void* d, int v, size_t n, void*) { memset(d, v, n); return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipSetDevice(int) { return 0; }
int hipGetLastError() { return 0; }
int hipDeviceSynchronize() { return 0; }
int hipGetSymbolAddress(void** p, const void*) { static double a[1 << 23]; *p = a; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 1; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipEventCreate(void** e) { *e = malloc(1); return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = malloc(1); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { *s = malloc(1); return 0; }
int hipStreamDestroy(void* s) { free(s); return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamIsCapturing(void*, int* c) { *c = capturing; return 0; }
int hipThreadExchangeStreamCaptureMode(int*) { return 0; }
struct Dim { unsigned x, y, z; };
static Dim cfg[2];
static std::map<const void*, const char*> names;
static char trail[1 << 16];
// the launches since the last call, "kernel grid threads;" each
const char* shim_launches() { static char out[1 << 16]; strcpy(out, trail); trail[0] = 0; return out; }
static char last_kernel[512];
static unsigned last_threads;
static float (*timer)(const char*, unsigned) = nullptr;
void shim_timer(float (*f)(const char*, unsigned)) { timer = f; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = timer ? timer(last_kernel, last_threads) : 1.0f; return 0; }
int hipLaunchKernel(const void* f, Dim g, Dim b, void**, size_t, void*) {
  snprintf(last_kernel, sizeof last_kernel, "%s", names.count(f) ? names[f] : "?");
  last_threads = b.x;
  const size_t n = strlen(trail);
  snprintf(trail + n, sizeof trail - n, "%s %u %u;", last_kernel, g.x, b.x);
  return 0;
}
int __hipPushCallConfiguration(Dim g, Dim b, size_t, void*) { cfg[0] = g; cfg[1] = b; return 0; }
int __hipPopCallConfiguration(Dim* g, Dim* b, size_t* m, void** s) { *g = cfg[0]; *b = cfg[1]; *m = 0; *s = nullptr; return 0; }
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { names[f] = name; }
}
"""

# (the layout of the properties is the runtime's own)
PROPERTIES = r"""
#include <cstring>
#include <hip/hip_runtime_api.h>
extern "C" hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_t* p, int) {
  memset((void*)p, 0, sizeof *p);
  strcpy(p->gcnArchName, "gfx950:test");
  return hipSuccess;
}
"""

PRELUDE = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
shim.shim_used.restype = ctypes.c_size_t
shim.shim_launches.restype = ctypes.c_char_p
shim.shim_budget.argtypes = [ctypes.c_size_t]
sys.path.insert(0, sys.argv[2])
import meshgen as mg
from paper_2508_17917_amd import _lib as L
lib = L.load()

def context(p, nt, nr, precision=0, mesh=None):
    m = mesh or mg.ogrid(nt, nr, 0.5, 5.0, 1.02)
    h = L.dg_create(p, precision)
    L.dg_set_physics(h, 1.4, 0.72, 1e-3, 1.0, 0, 1.0, [1, 0.2, 0, 1.8])
    L.dg_set_mesh(h, m["VX"], m["VY"], m["EToV"], m["face_tag"], m["period"])
    L.dg_setup(h)
    return h

def state(p, K):
    return K * 4 * ((p + 1) * (p + 2) // 2) * 8

def trace(p, K, size=8):
    return K * 3 * (p + 1) * 4 * size

def buffers(n):
    return [ctypes.create_string_buffer(n) for _ in range(2)]

VW = (ctypes.c_double * 2)(0.0, 0.0)
"""


def _child(tmp_path, body):
    so, script = str(tmp_path / "shim.so"), str(tmp_path / "child.py")
    rocm = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")
    objs = []
    for name, text in (("shim", SHIM), ("properties", PROPERTIES)):
        path = str(tmp_path / (name + ".cpp"))
        with open(path, "w") as fh:
            fh.write(text)
        objs.append(str(tmp_path / (name + ".o")))
        subprocess.run(["g++", "-O1", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", rocm, "-c", "-o", objs[-1], path], check=True)
    subprocess.run(["g++", "-shared", "-o", so] + objs, check=True)
    with open(script, "w") as fh:
        fh.write(PRELUDE + body)
    r = subprocess.run([sys.executable, script, so, ROOT], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("done"), r.stdout + r.stderr


def test_a_batch_needs_no_more_than_its_states(tmp_path):
    """Room for the states and tables and most of the traces: the batch is made
    (from its states); with ample room it takes the traces, and gives all back."""
    _child(tmp_path, r"""
hs = [context(3, 97, 60), context(1, 83, 41)]
Ks = [L.dg_num_elements(h) for h in hs]
assert sum(Ks) >= 16384
states = sum(3 * state(p, K) for p, K in zip((3, 1), Ks))
traces = sum(2 * trace(p, K) for p, K in zip((3, 1), Ks))
before = shim.shim_used()
b = L.dg_batch_create(hs)
took = shim.shim_used() - before
assert states + traces <= took <= states + traces + 65536, (took, states, traces)
L.dg_batch_destroy(b)
assert shim.shim_used() == before
shim.shim_budget(before + states + 65536 + traces * 9 // 10)
b = L.dg_batch_create(hs)
assert states <= shim.shim_used() - before <= states + 65536
L.dg_batch_destroy(b)
assert shim.shim_used() == before
shim.shim_budget(before + states // 2)
try:
    L.dg_batch_create(hs)
    raise SystemExit("a batch beyond the memory was made")
except L.DGError as e:
    assert e.code == L.DG_ENOMEM
assert shim.shim_used() == before
print("done")
""")


def test_a_context_takes_step_memory_with_its_first_steps(tmp_path):
    """Set-up takes none; a captured call takes none and fails nothing; the first
    plain call takes the traces and, for an odd number of steps, the second
    scratch state; a switch to over-integration takes its larger traces; where
    that would leave less than half of the free memory, nothing is taken and the
    steps run all the same."""
    _child(tmp_path, r"""
base0 = shim.shim_used()
h = context(4, 67, 64)
K = L.dg_num_elements(h)
S, T, TOI = state(4, K), trace(4, K), K * 3 * 7 * 8 * 8
set_up = shim.shim_used()
# geometry, connectivity and the CFL work per element, one state, operators
assert set_up - base0 <= K * (128 + 12 + 48) + S + (1 << 20), set_up - base0
U, K1 = buffers(S)
F = ctypes.create_string_buffer(24 * 8)

def steps(n, h=h, U=U, K1=K1):
    assert lib.dg_rk_steps(h, U, K1, n, 1e-6, VW, F, None) == 0, L.dg_last_error(h)

shim.shim_capturing(1)
steps(3)
assert lib.dg_rk_step(h, U, K1, 1e-6, VW, None) == 0
shim.shim_capturing(0)
assert shim.shim_used() == set_up
assert lib.dg_rk_step(h, U, K1, 1e-6, VW, None) == 0   # one step of 8,576 elements: no traces
assert shim.shim_used() == set_up + S
steps(2)
assert shim.shim_used() == set_up + S + 2 * T
steps(3)
assert shim.shim_used() == set_up + S + 2 * T
L.dg_set_overintegration(h, 1)
steps(2)
assert shim.shim_used() == set_up + S + 2 * T + 2 * TOI
L.dg_set_overintegration(h, 0)
steps(2)
assert shim.shim_used() == set_up + S + 2 * T + 2 * TOI
L.dg_destroy(h)
assert shim.shim_used() == base0

h = context(4, 67, 64)
for room in (S + S // 2, 2 * S + T):
    shim.shim_budget(shim.shim_used() + room)
    for n in (3, 2):
        before = shim.shim_used()
        steps(n, h)
        assert shim.shim_used() - before <= room // 2
# a refusal stands until the next set-up
shim.shim_budget(1 << 40)
before = shim.shim_used()
steps(3, h)
assert shim.shim_used() == before
L.dg_setup(h)
steps(3, h)
assert shim.shim_used() == set_up + S + 2 * T
L.dg_destroy(h)
assert shim.shim_used() == base0
print("done")
""")


def test_a_batch_takes_traces_where_they_pay(tmp_path):
    """From 16,384 elements on; where all instances are of order 3 or 4, 32,768."""
    _child(tmp_path, r"""
small, large = mg.ogrid(91, 45, 0.5, 5.0, 1.02), mg.ogrid(97, 86, 0.5, 5.0, 1.02)   # 8,190 and 16,684
def traces(*what):
    hs = [context(p, 0, 0, f, m) for p, m, f in what]
    Ks = [L.dg_num_elements(h) for h in hs]
    before = shim.shim_used()
    b = L.dg_batch_create(hs)
    extra = shim.shim_used() - before - sum(3 * state(p, K) for (p, m, f), K in zip(what, Ks))
    L.dg_batch_destroy(b)
    want = sum(2 * trace(p, K, 4 if f == 2 else 8) for (p, m, f), K in zip(what, Ks))
    for h in hs:
        L.dg_destroy(h)
    assert extra < 65536 or want <= extra < want + 65536
    return extra >= 65536
for f in (0, 2):
    for p in (1, 2, 5, 6):
        assert not traces((p, small, f), (p, small, f)) and traces((p, large, f))
    for p in (3, 4):
        assert not traces((p, large, f), (p, small, f)) and traces((p, large, f), (7 - p, large, f))
        assert traces((p, small, f), (2, large, f))
assert not traces((4, large, 3), (4, large, 3))   # bfloat16 operators
print("done")
""")
