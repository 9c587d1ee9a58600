"""Device code compiled for the host, to be called from a test program: headers of the library with the built-ins they use defined in plain C++.  (Without the
signed arithmetic for primes just below 2^60, which is written with an instruction of its own.)"""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_09424_amd", "csrc")

PREAMBLE = r"""
#include <cmath>
#include <cstdio>
#include <cstring>
#include <hip/hip_runtime.h>
#define __launch_bounds__(...)
#define HIP_DYNAMIC_SHARED(type, name) extern type name[];
#define __builtin_amdgcn_sbfe(x, o, w) ((int)((x) << (32 - (w) - (o))) >> (32 - (w)))
#define __builtin_amdgcn_fence(...)
#define __builtin_amdgcn_wave_barrier()
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_sched_barrier(x)
static struct { unsigned x, y, z; } threadIdx, blockIdx;
static inline double __longlong_as_double(long long x) { double d; memcpy(&d, &x, 8); return d; }
static inline long long __double_as_longlong(double d) { long long x; memcpy(&x, &d, 8); return x; }
static inline unsigned long long __umul64hi(unsigned long long a, unsigned long long b) { return (unsigned __int128)a * b >> 64; }
static inline unsigned __brev(unsigned x) { unsigned r = 0; for (int i = 0; i < 32; i++) r |= (x >> i & 1) << (31 - i); return r; }
static inline int __clz(unsigned x) { return __builtin_clz(x); }
static inline void __syncthreads() {}
#include "keyswitch16_kernels.h"
"""


def run(tmp_path, program):
    """Compiles a program after the preamble, runs it and returns the numbers it prints."""
    src, exe = tmp_path / "host.cpp", tmp_path / "host"
    src.write_text(PREAMBLE + program)
    subprocess.run(["g++", "-O1", "-ffp-contract=off", "-std=c++17", "-w", "-fpermissive", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC, str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return [[float(x) for x in line.split()] for line in r.stdout.splitlines()]
