"""Launch shapes and the autotuner on the CPU: which kernels run in which shape,
seen by a stand-in for the runtime's calls (tests/test_memory_host.py) that
keeps a list of the launches and gives the times that the tuner reads.
"""
from tests.test_memory_host import _child, pytestmark  # noqa: F401

SHAPES = r"""
import re
U, K1 = buffers(state(6, 20000))
F = ctypes.create_string_buffer(24 * 16)

def launches(call):
    shim.shim_launches()
    call()
    out = []
    for line in shim.shim_launches().decode().split(";")[:-1]:
        name, grid, threads = line.split()
        out.append((re.sub(r"^_ZN4dgmi\d+", "", name), int(grid), int(threads)))
    return out

def rhs(h):
    return launches(lambda: L._check(lib.dg_rhs(h, U, K1, VW, None), h))

def steps(h, n=2):
    return launches(lambda: L._check(lib.dg_rk_steps(h, U, K1, n, 1e-6, VW, None, None), h))

def tune(h, path=None):
    best = ctypes.c_double()
    L._check(lib.dg_autotune(h, U, 2, path, None, ctypes.byref(best)), h)
    return best.value

def threads_of(ls, kernel):
    got = {t for n, g, t in ls if n.startswith(kernel)}
    assert len(got) == 1, (kernel, ls)
    return got.pop()
"""


def test_each_kernel_gets_its_own_shape(tmp_path):
    """A timer on which the stage from the states is faster with four waves and the
    one from traces with two: each runs with its own, also from the cache; a
    line without the kernel's name, of the other kernel or of curved elements is
    not taken."""
    _child(tmp_path, SHAPES + r"""
import json
FN = ctypes.CFUNCTYPE(ctypes.c_float, ctypes.c_char_p, ctypes.c_uint)
fast = {True: 128, False: 256}
timer = FN(lambda name, threads: 1.0 if threads == fast[b"trace" in name] else 2.0)
shim.shim_timer(timer)
path = sys.argv[1].replace("shim.so", "tune.jsonl").encode()
old = '{"arch": "gfx950:test", "p": 4, "precision": 2, "K": 8576, "waves": 4, "grid": 3, "us": 11.000}\n'
open(path, "w").write(old)
h = context(4, 67, 64, precision=2)
assert tune(h, path) > 0.0
lines = open(path).read().splitlines()
assert len(lines) == 2
line = json.loads(lines[1])
assert (line["kernel"], line["curved"], line["waves"], line["stage_waves"]) == ("traces", 0, 2, 4), line
assert threads_of(steps(h), "trace_stage_kernel") == 128
assert threads_of(rhs(h), "stage_kernel") == 256
assert L.dg_get_tuning(h)[0] == 2
fast = {True: 256, False: 128}   # not asked: the line serves
h2 = context(4, 67, 64, precision=2)
assert tune(h2, path) == 0.0
assert threads_of(steps(h2), "trace_stage_kernel") == 128 and threads_of(rhs(h2), "stage_kernel") == 256
assert steps(h2) == steps(h) and rhs(h2) == rhs(h)
# bfloat16 operators have no traces, and another precision: a line of its own
hb = context(4, 67, 64, precision=3)
assert tune(hb, path) > 0.0
assert json.loads(open(path).read().splitlines()[-1])["kernel"] == "states"
assert threads_of(steps(hb), "stage_kernel") == threads_of(rhs(hb), "stage_kernel") == 128
# the same order and precision without memory for traces
n = len(open(path).read().splitlines())
hn = context(4, 67, 64, precision=2)
shim.shim_budget(shim.shim_used() + 2 * trace(4, 8576, 4))
assert tune(hn, path) > 0.0
shim.shim_budget(1 << 40)
lines = [json.loads(x) for x in open(path).read().splitlines()[n:]]
assert len(lines) == 1 and lines[0]["kernel"] == "states" and lines[0]["waves"] == lines[0]["stage_waves"] == 2
h3 = context(4, 67, 64, precision=2)
assert tune(h3, path) == 0.0 and L.dg_get_tuning(h3)[0] == 2
print("done")
""")


def test_the_reported_shape_changes_nothing(tmp_path):
    """dg_set_tuning(dg_get_tuning()) on every order and form, nodal and over-
    integrated, on meshes that fill the chip and that do not: the same launches
    of right-hand sides and steps as before, by default, after a shape was set
    and after the autotuner picked one a kernel.  Another shape does change them."""
    _child(tmp_path, SHAPES + r"""
FN = ctypes.CFUNCTYPE(ctypes.c_float, ctypes.c_char_p, ctypes.c_uint)
timer = FN(lambda name, threads: 1.0 if threads == (128 if b"trace" in name else 256) else 2.0)
shim.shim_timer(timer)
for nt, nr in ((9, 5), (101, 99)):
    mesh = mg.ogrid(nt, nr, 0.5, 5.0, 1.01)
    for p, precision, oi in [(p, f, 0) for p in (1, 4, 6) for f in (0, 2, 3)] + [(p, 0, 1) for p in (3, 4, 5)]:
        h = context(p, nt, nr, precision, mesh)
        L.dg_set_overintegration(h, oi)
        big = buffers(state(p, 2 * nt * nr))
        U, K1 = big
        for how in ("default", "set", "tuned"):
            if how == "set":
                L.dg_set_tuning(h, 2, 1)
                assert L.dg_get_tuning(h) == (2, 1)
            if how == "tuned":
                tune(h)
            before = rhs(h), steps(h)
            L.dg_set_tuning(h, *L.dg_get_tuning(h))
            assert (rhs(h), steps(h)) == before, (nt, p, precision, oi, how)
        if oi and nr == 99:
            L.dg_set_tuning(h, 0, 0)
            w = L.dg_get_tuning(h)[0]
            default = steps(h)
            L.dg_set_tuning(h, 6 - w, 0)   # the other of 2 and 4
            assert steps(h) != default
        L.dg_destroy(h)
print("done")
""")
