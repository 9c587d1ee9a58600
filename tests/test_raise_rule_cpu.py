"""Which form of raised digits a call's rotations read, and that the form without row passes is not taken for groups."""
import os
import subprocess

from paper_2509_09424_amd import binding

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_09424_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "api_util.h"
#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main() {
    // a group of two on one raised ciphertext, by way of the rule and past it; refused before the device is touched
    ensi_ctx ctx;
    ctx.ks16 = true;
    CHECK(run_rotations(&ctx, nullptr, 2, 3, 3, 3, RAISE_ONE, nullptr, 2) == ENSI_E_BADARG);
    CHECK(raise_use(2, 1, 2) == RAISE_SHARED && raise_use(3, 1, 3) == RAISE_SHARED);
    CHECK(raise_use(1, 1) == RAISE_ONE && raise_use(2, 1) == RAISE_ONE && raise_use(3, 1) == RAISE_SHARED);
    CHECK(raise_use(32, 16) == RAISE_ONE && raise_use(33, 16) == RAISE_SHARED);
    fflush(stdout);
    _Exit(0);  // (the context was never opened on a device)
}
"""


def test_groups_never_read_digits_without_their_row_passes(tmp_path):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(PROGRAM)
    lib = os.path.dirname(binding.LIB_PATH)
    subprocess.run(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC, str(src), "-o", str(exe), binding.LIB_PATH,
                    "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath," + lib + ":/opt/rocm/lib"], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
