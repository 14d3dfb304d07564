"""What a step does whose recording as a graph fails: the library's own host code over a stand-in for the HIP runtime (no
GPU, kernels do nothing, a chosen function fails), in a process of its own."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
_RUNTIME = r"""
#include <stdlib.h>
#include <string.h>
enum { OUT_OF_MEMORY = 2, CAPTURE_INVALID = 901 };
int launches, recorded, captures, graphs, replays, capturing, last_error;   /* graphs: alive */
const char *fail_in = "";                                                   /* the function that fails */
static int fails(const char *f, int code) { return !strcmp(f, fail_in) ? (last_error = code) : 0; }
int hipGetLastError(void) { int e = last_error; last_error = 0; return e; }
const char *hipGetErrorString(int e) { return "an error"; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int what, int d) { *v = 8; return 0; }
int hipMalloc(void **p, size_t n) { *p = calloc(n + 16, 1); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned f) { return hipMalloc(p, n); }
int hipFree(void *p) { free(p); return 0; }
int hipHostFree(void *p) { free(p); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int k) { memmove(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { memmove(d, s, n); return 0; }
int hipMemsetAsync(void *p, int v, size_t n, void *st) { memset(p, v, n); return 0; }
int hipStreamSynchronize(void *st) { return 0; }
int hipEventCreate(void **e) { *e = 0; return 0; }
int hipEventDestroy(void *e) { return 0; }
int hipEventRecord(void *e, void *st) { return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { *ms = 0; return 0; }
int hipGetSymbolAddress(void **p, const void *s) { *p = 0; return 1; }
int hipStreamBeginCapture(void *st, int mode) {
    if (fails("begin", OUT_OF_MEMORY)) return OUT_OF_MEMORY;
    ++captures; capturing = 1; return 0;
}
int hipStreamEndCapture(void *st, void **g) {
    capturing = 0; *g = 0;
    if (fails("end", CAPTURE_INVALID)) return CAPTURE_INVALID;
    *g = malloc(1); ++graphs; return 0;
}
int hipGraphInstantiate(void **e, void *g, void *node, char *log, size_t n) {
    if (fails("instantiate", OUT_OF_MEMORY)) { *e = (void *)1; return OUT_OF_MEMORY; }
    *e = malloc(1); return 0;
}
int hipGraphLaunch(void *e, void *st) { if (fails("replay", OUT_OF_MEMORY)) return OUT_OF_MEMORY; ++replays; return 0; }
int hipGraphDestroy(void *g) { --graphs; free(g); return 0; }
int hipGraphExecDestroy(void *e) { free(e); return 0; }
typedef struct { unsigned x, y, z; } dim3_t;
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t shm, void *st) { return 0; }
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *shm, void **st) { *g = *b = (dim3_t){1, 1, 1}; *shm = 0; *st = 0; return 0; }
int hipLaunchKernel(const void *f, dim3_t g, dim3_t b, void **args, size_t shm, void *st) {
    if (!capturing) ++launches;
    else if (fails("record", CAPTURE_INVALID)) return CAPTURE_INVALID;
    else ++recorded;
    return 0;
}
static void *binary;
void **__hipRegisterFatBinary(const void *d) { return &binary; }
void __hipUnregisterFatBinary(void **m) {}
void __hipRegisterFunction(void) {}
void __hipRegisterVar(void) {}
"""
_CHILD = r"""
import ctypes as C, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[3])
import paper_2512_07503_amd as sjd
from paper_2512_07503_amd.binding import ModelDesc, Weights, Sampling, StepResult
L = sjd.lib()
def n(name): return C.c_int.in_dll(fake, name).value
one = (C.c_char * (1 << 20))()
p = C.cast(one, C.c_void_p)
arr = C.cast((C.c_void_p * 2)(p.value, p.value), C.POINTER(C.c_void_p))
w = Weights(p, p, p, *[arr] * 9)
md = ModelDesc(2, 128, 2, 2, 128, 64, 0, 64, 1e-5, 1e4, int(sys.argv[4]), 1, 64, 4, 0, 0)
ctx, stream = C.c_void_p(), C.c_void_p(C.addressof(one))
assert L.sjd_create(C.byref(md), C.byref(w), C.byref(Sampling(3.0, 1.0, 10, 0.5, 0, 0, 0)), stream, C.byref(ctx)) == 0, L.sjd_last_error(None)
ids = (C.POINTER(C.c_int32) * 1)((C.c_int32 * 3)(1, 2, 3))
len3, n_img = (C.c_int32 * 1)(3), (C.c_int32 * 1)(20)
assert L.sjd_prefill(ctx, 1, ids, len3, ids, len3, n_img) == 0
res = (StepResult * 1)()
fail_in = C.create_string_buffer(sys.argv[2].encode())
C.c_void_p.in_dll(fake, "fail_in").value = C.addressof(fail_in)
codes, launched = [], []
for _ in range(4):
    before = n("launches")
    codes.append(L.sjd_step(ctx, res))
    launched.append(n("launches") - before)
print(repr(dict(codes=codes, launched=launched, captures=n("captures"), graphs=n("graphs"), replays=n("replays"))))
L.sjd_destroy(ctx)
print(n("graphs"))
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    d = tmp_path_factory.mktemp("runtime")
    (d / "runtime.c").write_text(_RUNTIME)
    graph = ["hipStreamBeginCapture", "hipStreamEndCapture", "hipGraphInstantiate", "hipGraphLaunch", "hipGraphDestroy", "hipGraphExecDestroy"]
    (d / "versions").write_text("hip_4.2 { global: *; };\nhip_4.3 { global: %s; };\n" % "; ".join(graph))
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", "-O1", str(d / "runtime.c"), "-o", str(d / "runtime.so"),
                    "-Wl,-soname,libamdhip64.so.7", f"-Wl,--version-script,{d / 'versions'}"], check=True)
    return d / "runtime.so"


def _run(runtime, fail_in, dtype):
    r = subprocess.run([sys.executable, "-c", _CHILD, str(runtime), fail_in, ROOT, str(dtype)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    seen, left = r.stdout.splitlines()
    assert int(left) == 0                       # every graph is destroyed with its context, if not before
    return eval(seen)


@pytest.mark.parametrize("dtype", [0, 1])
def test_recorded_steps_are_replayed(runtime, dtype):
    s = _run(runtime, "", dtype)
    assert s["codes"] == [0] * 4 and s["launched"][0] > 10 and s["launched"][1:] == [0] * 3
    assert s["captures"] == 1 and s["replays"] == 3 and s["graphs"] == 1


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("fail_in", ["begin", "record", "end", "instantiate"])
def test_a_step_whose_recording_fails_is_a_step(runtime, fail_in, dtype):
    """The launches have run by then: the step succeeds, nothing is recorded again, and the steps after it are launched kernel by
    kernel, undisturbed by the error that the runtime keeps for whoever asks next."""
    s = _run(runtime, fail_in, dtype)
    assert s["codes"] == [0] * 4 and s["launched"][0] > 10 and s["launched"] == [s["launched"][0]] * 4
    assert s["captures"] <= 1 and s["replays"] == 0 and s["graphs"] == 0


def test_a_replay_that_fails_has_run_nothing(runtime):
    s = _run(runtime, "replay", 1)
    assert s["codes"][0] == 0 and s["codes"][1:] == [-4] * 3 and s["launched"][1:] == [0] * 3
