"""Which kernels a signed sum takes."""
import os
import subprocess

import pytest

import simhip
from paper_2509_09424_amd import binding

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_09424_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "common.h"
// operands, outputs, mode, rescale, the code that the call has to return
int main(int, char **v) {
    const int n_v = atoi(v[1]), m = atoi(v[2]), mode = atoi(v[3]), rescale = atoi(v[4]);
    ensi_ctx ctx;
    ctx.N = 4096;
    ctx.primes.assign(ENSI_MAX_EXT, 97);
    const int nk = (n_v + 255) / 256 * 256;
    double fc = 0;
    const int code = launch_accumulate_mfma(&ctx, nullptr, 0, n_v, nk, nullptr, nullptr, nullptr, 7, mode, m, 2, 2 + rescale, nullptr, 2, rescale ? &fc : nullptr, nullptr);
    _Exit(code != atoi(v[5]));
}
"""
POS7, FP8, INT8 = 0, 1, 2


@pytest.fixture(scope="module")
def product(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("rule")
    (tmp / "rule.cpp").write_text(PROGRAM)
    lib = os.path.dirname(binding.LIB_PATH)
    subprocess.run(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC, str(tmp / "rule.cpp"), "-o", str(tmp / "rule"), binding.LIB_PATH,
                    "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath," + lib + ":/opt/rocm/lib"], check=True)

    def run(n_v, m, mode, rescale, code=0):
        calls = simhip.run(tmp, command=[str(a) for a in (tmp / "rule", n_v, m, mode, rescale, code)])
        return [c[2] for c in calls if c[0] == "launch"]
    return run


@pytest.mark.parametrize("n_v,m", [(300, 300), (64, 64), (384, 4096), (4096, 384)])
def test_weights_of_never_negative_digits_never_meet_signed_ones(product, n_v, m):
    """Weights prepared for AM_POS7 are plus one: read as signed ones the sums would be wrong without a word."""
    kernels = product(n_v, m, POS7, 0)
    assert kernels and not any("direct" in k for k in kernels) and any("k_word_sums" in k for k in kernels), kernels


def test_fused_rescale_of_wide_primes_is_refused(product):
    """It would launch nothing, or work in double precision on residues that do not fit it."""
    for n_v in (64, 600):
        assert product(n_v, 64, INT8, 1, code=-1) == []
