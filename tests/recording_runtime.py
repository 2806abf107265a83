"""A stand-in for the HIP runtime that records what the library asks of it: host code that needs a device (uploads, choice of kernels,
their grids) and its failures are then checked without one.  Kernels do not run and nothing is copied.

`record(tmp, script)` runs `script` in a child process, in which `sb` is the binding, `fake(n)` an address that stands for n bytes
on the device, `log()` the calls since the last `log()` and `fail(name, nth)` makes the nth call of a function from now on
fail, and returns what the script gives to `answer(value)`."""
import json
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <hip/hip_runtime_api.h>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
static std::string text, last;
static std::map<const void *, std::string> names;
static std::map<std::string, int> failing;
static int cus = 256, sramecc = 1;
static struct { dim3 g, b; size_t lds; hipStream_t s; } cfg;
static hipError_t did(const char *name)
{
    auto f = failing.find(name);
    return f != failing.end() && --f->second == 0 ? hipErrorOutOfMemory : hipSuccess;
}
extern "C" {
void recorder_device(int c, int ecc) { cus = c; sramecc = ecc; }
void recorder_fail(const char *name, int nth) { failing[name] = nth; }
const char *recorder_log() { last = text; text.clear(); return last.c_str(); }
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *, int *) { names[f] = name; }
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) { cfg = {g, b, lds, s}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s) { *g = cfg.g; *b = cfg.b; *lds = cfg.lds; *s = cfg.s; return hipSuccess; }
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t lds, hipStream_t)
{
    char line[1024];
    snprintf(line, sizeof line, "launch %s grid %u,%u,%u block %u lds %zu\n", names[f].c_str(), g.x, g.y, g.z, b.x, lds);
    text += line;
    return did("hipLaunchKernel");
}
hipError_t hipMemcpyAsync(void *, const void *src, size_t n, hipMemcpyKind kind, hipStream_t)
{
    char line[64];
    unsigned long long h = 14695981039346656037ull;
    if (kind == hipMemcpyHostToDevice)
        for (size_t i = 0; i < n; ++i) h = (h ^ ((const unsigned char *)src)[i]) * 1099511628211ull;
    snprintf(line, sizeof line, "copy %zu %llx\n", n, h);
    text += line;
    return did("hipMemcpyAsync");
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    const hipError_t e = did("hipHostMalloc");
    *p = e == hipSuccess ? calloc(1, n) : nullptr;
    return e;
}
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *ev, unsigned)
{
    const hipError_t e = did("hipEventCreateWithFlags");
    if (e == hipSuccess) { *ev = (hipEvent_t)malloc(8); text += "event made\n"; }
    return e;
}
hipError_t hipEventDestroy(hipEvent_t ev) { free((void *)ev); text += "event gone\n"; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return did("hipEventRecord"); }
hipError_t hipEventSynchronize(hipEvent_t) { return did("hipEventSynchronize"); }
hipError_t hipStreamSynchronize(hipStream_t) { return did("hipStreamSynchronize"); }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { *p = (void *)4096; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = cus; return hipSuccess; }
#undef hipGetDeviceProperties
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = cus;
    snprintf(p->gcnArchName, sizeof p->gcnArchName, "gfx950:sramecc%c:xnack-", sramecc ? '+' : '-');
    return hipSuccess;
}
}
"""

PRELUDE = r"""
import ctypes, json, sys
rec = ctypes.CDLL(%r, mode=ctypes.RTLD_GLOBAL)             # before the library: its calls are bound to the first that has them
rec.recorder_log.restype = ctypes.c_char_p
log = lambda: rec.recorder_log().decode().splitlines()
fail = lambda name, nth=1: rec.recorder_fail(name.encode(), nth)
device = rec.recorder_device
_at = [1 << 40]
def fake(n):
    _at[0] += (int(n) + 4095) // 4096 * 4096
    return _at[0] - (int(n) + 4095) // 4096 * 4096
def answer(value):
    print("ANSWER " + json.dumps(value))
from paper_2602_17698_amd import binding as sb
"""


def record(tmp, script):
    cxx = shutil.which("g++")
    include = "/opt/rocm/include"
    if cxx is None or not os.path.exists(include):
        pytest.skip("needs g++ and the HIP headers")
    lib = str(tmp / "librecorder.so")
    (tmp / "recorder.cpp").write_text(SOURCE)
    subprocess.check_call([cxx, "-std=c++17", "-O1", "-w", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I" + include, "-o", lib,
                           str(tmp / "recorder.cpp")])
    r = subprocess.run([sys.executable, "-c", PRELUDE % lib + script], cwd=ROOT, stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                       text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-3000:]
    return json.loads([line for line in r.stdout.splitlines() if line.startswith("ANSWER ")][-1][7:])
