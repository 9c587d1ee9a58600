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
// operands, outputs, mode, rescale, the code that the call has to return, ring, limbs, planes
int main(int, char **v) {
    const int n_v = atoi(v[1]), m = atoi(v[2]), mode = atoi(v[3]), rescale = atoi(v[4]), limbs = atoi(v[7]);
    ensi_ctx ctx;
    ctx.N = 1 << atoi(v[6]);
    ctx.primes.assign(ENSI_MAX_EXT, 97);
    const int nk = (n_v + 255) / 256 * 256;
    double fc = 0;
    const int code = launch_accumulate_mfma(&ctx, nullptr, 0, n_v, nk, nullptr, nullptr, nullptr, atoi(v[8]), mode, m, limbs, limbs + rescale, nullptr, limbs, rescale ? &fc : nullptr, nullptr);
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

    def run(n_v, m, mode, rescale, code=0, ring=12, limbs=2, planes=7):
        calls = simhip.run(tmp, command=[str(a) for a in (tmp / "rule", n_v, m, mode, rescale, code, ring, limbs, planes)])
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


@pytest.mark.parametrize("ring,limbs,planes,n_v,m,rescale,direct", [
    # fewer word tiles than the 256 CUs: a block runs through all outputs while other CUs have none
    (10, 2, 7, 256, 384, 0, True), (10, 2, 7, 256, 1024, 0, False), (10, 2, 7, 384, 2048, 0, False), (10, 2, 5, 16, 960, 0, True), (10, 2, 5, 16, 2048, 0, False),
    (10, 2, 7, 8, 512, 1, True), (10, 2, 7, 8, 4096, 1, False), (7, 2, 5, 4096, 384, 0, False), (10, 2, 7, 4096, 384, 0, False), (10, 2, 7, 768, 8, 0, True),
    # blocks that take a CU each, in a last round that leaves half of them empty
    (11, 3, 7, 384, 1024, 0, False), (11, 3, 5, 384, 1024, 0, True), (12, 2, 7, 384, 1024, 0, True), (11, 3, 7, 256, 1024, 0, True), (12, 3, 5, 256, 4096, 0, False),
    # many outputs
    (16, 16, 7, 384, 3072, 0, True), (16, 16, 7, 384, 4096, 0, False), (16, 16, 7, 256, 4096, 0, True), (16, 8, 5, 384, 4096, 0, True), (16, 16, 7, 128, 4096, 1, True),
    # few outputs of many operands
    (12, 2, 7, 4096, 384, 0, True), (16, 16, 7, 4096, 384, 0, True), (16, 16, 7, 4096, 385, 0, False), (16, 16, 7, 129, 8, 1, False)])
def test_digits_stay_in_lds_where_that_is_faster(product, ring, limbs, planes, n_v, m, rescale, direct):
    kernels = product(n_v, m, FP8, rescale, ring=ring, limbs=limbs, planes=planes)
    assert ("k_accumulate_direct" in kernels[0]) == direct and (len(kernels) == 1) == direct, kernels
