"""A step's two streams wait for each other's kernels through events, most of them bound to a kernel's launch.
A launch or a record that fails leaves its event where it was; whatever waits for it then starts too early.
Here libmimose runs on a stand-in for the HIP runtime that launches nothing, on host memory, without a GPU, and
fails one marking of an event after the other: the step has to return the error, wait for no such event, and
leave nothing behind that a later step reports."""
import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# entry points of the HIP runtime that the library calls, found here before those of the real one
RUNTIME = r"""
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>
struct dim3 { unsigned x, y, z; };
static long next_event = 1, marks = 0, fail_at = -1;
static void* bad = nullptr;                 // the event whose marking failed
static int bad_waits = 0, last_error = 0, error_code = 719;
static int mark(void* ev) {
  if (!ev) return 0;
  if (marks++ == fail_at) { bad = ev; return last_error = error_code; }
  if (ev == bad) bad = nullptr;
  return 0;
}
extern "C" {
void shim_fail_at(long n) { marks = 0; fail_at = n; bad = nullptr; bad_waits = 0; }
long shim_marks() { return marks; }
int shim_bad_waits() { return bad_waits; }
int hipEventCreate(void** e) { *e = (void*)next_event++; return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = (void*)next_event++; return 0; }
int hipEventDestroy(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 0.01f; return 0; }
int hipEventRecord(void* e, void*) { return mark(e); }
int hipEventSynchronize(void*) { return 0; }
int hipStreamWaitEvent(void*, void* e, unsigned) { if (e == bad) ++bad_waits; return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { *s = (void*)next_event++; return 0; }
int hipStreamDestroy(void*) { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int) { return "stand-in"; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return 0; }
int hipHostFree(void* p) { free(p); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { memcpy(d, s, n); return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int __hipPushCallConfiguration(dim3, dim3, size_t, void*) { return 0; }
int __hipPopCallConfiguration(dim3* a, dim3* b, size_t* n, void** s) { *a = *b = {1, 1, 1}; *n = 0; *s = nullptr; return 0; }
static std::map<const void*, std::string>& kernels() { static std::map<const void*, std::string> k; return k; }
static std::vector<const void*> launches;
void __hipRegisterFunction(void*, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { kernels()[host] = name; }
long shim_launches() { return (long)launches.size(); }
const char* shim_kernel(long i) { return kernels()[launches[i]].c_str(); }
int hipLaunchKernel(const void* k, dim3, dim3, void**, size_t, void*) { launches.push_back(k); return 0; }
int hipExtLaunchKernel(const void* k, dim3, dim3, void**, size_t, void*, void* start, void* stop, int) {
  launches.push_back(k);
  mark(start);
  return mark(stop);
}
}
"""

# a product without elements, with events
EMPTY = r"""
#include "kernels.h"
extern "C" int empty_product(void* gemm, void* start, void* stop) {
  mk::GemmArgs g{nullptr, 8, true, nullptr, 8, true, nullptr, 8, true, 0, 8, 8};
  g.time_start = (hipEvent_t)start;
  g.time_stop = (hipEvent_t)stop;
  return ((bool (*)(int, const mk::GemmArgs&, hipStream_t))gemm)(mk::BF16, g, nullptr);
}
"""

STEP = """
    import ctypes, sys
    runtime = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
    import numpy as np
    import paper_2209_02478_amd as mi
    import synthdata
    shape = synthdata.ModelShape(2, 128, 2, 256, 300, 96, sys.argv[2], causal=int(sys.argv[3]), pre_ln=int(sys.argv[3]),
                                 head=1 - int(sys.argv[3]))
    memory = np.zeros((64 << 20) + 256, np.uint8)
    ctx = mi.mimose_init(mi.make_cfg(synthdata.shape_dict(shape)), 0, (memory.ctypes.data + 255) // 256 * 256, 64 << 20)
    mi.mimose_force_plan(ctx, 0b01)
    mi.mimose_set_dropout(ctx, float(sys.argv[4]), 0.0, 5, 0)
    batch = synthdata.make_batch(shape, 4, 96, 3)
    assert batch[0].size * shape.hidden > 1 << 15                 # two streams
    runtime.shim_fail_at(ctypes.c_long(-1))
    mi.mimose_train_step(ctx, *batch, wait=False)
    n = runtime.shim_marks()
    assert n > 12, n
    for k in range(n):
        runtime.shim_fail_at(ctypes.c_long(k))
        try:
            mi.mimose_train_step(ctx, *batch, wait=False)
            raise SystemExit("marking %d of %d failed and the step did not say so" % (k, n))
        except mi.MimoseError as e:
            assert e.code == mi.MIMOSE_ERR_HIP, e
        assert runtime.shim_bad_waits() == 0, "a stream waits for marking %d of %d, which failed" % (k, n)
        runtime.shim_fail_at(ctypes.c_long(-1))
        mi.mimose_train_step(ctx, *batch, wait=True)
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    d = tmp_path_factory.mktemp("runtime")
    (d / "runtime.cpp").write_text(RUNTIME)
    (d / "empty.cpp").write_text(EMPTY)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", str(d / "runtime.so"), str(d / "runtime.cpp"),
                           str(d / "empty.cpp"), "-D__HIP_PLATFORM_AMD__", "-I" + os.environ.get("ROCM_PATH", "/opt/rocm") + "/include",
                           "-I" + os.path.join(ROOT, "paper_2209_02478_amd", "csrc")])
    return str(d / "runtime.so")


@pytest.mark.parametrize("dtype,pre_ln,p_drop", [("bf16", 0, 0.0), ("bf16", 0, 0.1), ("bf16", 1, 0.0), ("fp32", 0, 0.0), ("fp32", 1, 0.1)])
def test_failed_markings_reach_the_caller(runtime, dtype, pre_ln, p_drop):
    r = subprocess.run([sys.executable, "-c", textwrap.dedent(STEP), runtime, dtype, str(pre_ln), str(p_drop)], cwd=ROOT,
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


def test_empty_product_marks_its_events(runtime):
    """Whoever waits for a product's end waits for the event, also where there was nothing to launch."""
    code = """
        import ctypes, sys
        runtime = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
        import paper_2209_02478_amd as mi
        gemm = ctypes.cast(getattr(mi.load_library(), "_ZN2mk4gemmEiRKNS_8GemmArgsEP12ihipStream_t"), ctypes.c_void_p)
        for start, stop in ((0, 0), (0, 7), (6, 7)):
            runtime.shim_fail_at(ctypes.c_long(-1))
            assert runtime.empty_product(gemm, ctypes.c_void_p(start), ctypes.c_void_p(stop)) == 1
            assert runtime.shim_marks() == (start != 0) + (stop != 0), (start, stop, runtime.shim_marks())
    """
    r = subprocess.run([sys.executable, "-c", textwrap.dedent(code), runtime], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
