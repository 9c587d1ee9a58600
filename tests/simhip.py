"""A simulated HIP runtime: the runtime calls that the library imports, defined in a library of its own that is loaded first.  Device memory is host memory,
copies copy, kernels do not run; every call is written down with its stream, so that what a call launches, and in which order
the device may run it, can be checked without a GPU."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <hip/hip_runtime_api.h>
static FILE *log_file() {
    static FILE *f = fopen(getenv("SIMHIP_LOG"), "a");
    return f;
}
#define LOG(...) (fprintf(log_file(), __VA_ARGS__), fputc('\n', log_file()), fflush(log_file()))
static std::map<const void *, std::string> &names() { static std::map<const void *, std::string> m; return m; }
static struct { dim3 grid, block; size_t lds; hipStream_t st; } conf;
static int copies_until_failure = -1;
static hipError_t last = hipSuccess;
extern "C" {
void simhip_mark(const char *text) { LOG("mark %s", text); }
void simhip_fail_copy(int n) { copies_until_failure = n; }  // the asynchronous copy after n more fails
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { names()[f] = name; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t st) { conf = {g, b, lds, st}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *st) { *g = conf.grid; *b = conf.block; *lds = conf.lds; *st = conf.st; return hipSuccess; }
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t lds, hipStream_t st) {
    LOG("launch %p %s %u %u %zu", (void *)st, names()[f].c_str(), g.x * g.y * g.z, b.x, lds);
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_t *p, int) { memset(p, 0, sizeof *p); p->multiProcessorCount = 256; return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "simulated"; }
hipError_t hipGetLastError() { hipError_t e = last; last = hipSuccess; return e; }
hipError_t hipGetSymbolAddress(void **p, const void *) { static void *scratch = calloc(96, 1 << 20); *p = scratch; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { LOG("alloc"); *p = calloc(n ? n : 1, 1); return hipSuccess; }
hipError_t hipFree(void *p) { LOG("sync all"); free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { LOG("alloc"); *p = calloc(n, 1); return hipSuccess; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { LOG("sync (nil)"); memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpy2D(void *d, size_t dp, const void *s, size_t sp, size_t w, size_t h, hipMemcpyKind) {
    for (size_t i = 0; i < h; i++) memcpy((char *)d + i * dp, (const char *)s + i * sp, w);
    LOG("sync (nil)");
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st) {
    if (copies_until_failure >= 0 && copies_until_failure-- == 0) return hipErrorUnknown;
    LOG("copy %p %p %zu", (void *)st, d, n);
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemset(void *d, int v, size_t n) { memset(d, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t st) { LOG("fill %p", (void *)st); memset(d, v, n); return hipSuccess; }
hipError_t hipDeviceSynchronize() { LOG("sync all"); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *st, unsigned) { LOG("alloc"); *st = (hipStream_t)malloc(8); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t st) { free((void *)st); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t st) { LOG("sync %p", (void *)st); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t st, hipEvent_t e, unsigned) { LOG("wait %p %p", (void *)st, (void *)e); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { LOG("alloc"); *e = (hipEvent_t)malloc(8); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { free((void *)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t st) { LOG("record %p %p", (void *)st, (void *)e); return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { LOG("syncevent %p", (void *)e); return hipSuccess; }
hipError_t hipEventElapsedTime(float *t, hipEvent_t, hipEvent_t) { *t = 0; return hipSuccess; }
}
"""

PREAMBLE = """
import ctypes, os, sys
import numpy as np
sys.path.insert(0, %r)
from paper_2509_09424_amd import binding
sim = ctypes.CDLL(os.environ["SIMHIP"])
def mark(text): sim.simhip_mark(text.encode())
""" % ROOT


def run(tmp_path, body=None, command=None):
    """Runs a Python program, or a command, on the simulated runtime and returns what it called: a list of [what, stream, ...]."""
    src, lib, log, prog = tmp_path / "simhip.cpp", tmp_path / "libsimhip.so", tmp_path / "log", tmp_path / "prog.py"
    if not lib.exists():
        src.write_text(SOURCE)
        subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", str(src), "-o", str(lib)], check=True)
    if body is not None:
        prog.write_text(PREAMBLE + body)
        command = [sys.executable, str(prog)]
    log.write_text("")
    env = dict(os.environ, SIMHIP=str(lib), SIMHIP_LOG=str(log), LD_PRELOAD=str(lib) + ":" + os.environ.get("LD_PRELOAD", ""))
    r = subprocess.run(command, env=env, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return [line.split() for line in log.read_text().splitlines()]


def unordered(calls):
    """Pairs of device operations on different streams of which neither is ordered before the other, as indexes into calls.  Streams run in order;
    a wait orders what follows it after what the event had recorded; a host that has waited orders all that it enqueues later."""
    ops, host, stream, event = [], set(), {}, {}
    for k, c in enumerate(calls):
        what = c[0]
        if what in ("launch", "copy", "fill"):
            before = stream.setdefault(c[1], set()) | host
            ops.append((k, c[1], frozenset(before)))
            stream[c[1]] = before | {k}
        elif what == "record":
            event[c[2]] = set(stream.get(c[1], set()))
        elif what == "wait":
            stream[c[1]] = stream.get(c[1], set()) | event.get(c[2], set())
        elif what == "syncevent":
            host |= event.get(c[1], set())
        elif what == "sync":
            for st in stream if c[1] == "all" else [c[1]]:
                host |= stream.get(st, set())
    return [(i, k) for n, (k, st, before) in enumerate(ops) for i, other, _ in ops[:n] if other != st and i not in before]
