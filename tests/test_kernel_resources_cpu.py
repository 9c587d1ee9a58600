"""Registers of the kernels that hold whole rows or columns of a transform: what the compiler could not place goes through scratch
memory on every access, on the ring where it happens and nowhere else.  Read from the compiler's own report, ring by ring."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2509_09424_amd import build


def spilled(source):
    """{mangled kernel name: vector registers spilled} of one source (file, or file:ring as in the build's list)."""
    src, _, ring = source.partition(":")
    cmd = [build.HIPCC] + build.FLAGS + ["-DKS_RING=" + ring] * bool(ring) + ["-I" + os.path.join(build.CSRC, "inc"), "--cuda-device-only",
           "-Rpass-analysis=kernel-resource-usage", "-c", os.path.join(build.CSRC, src), "-o", os.devnull]
    report = subprocess.run(cmd, capture_output=True, text=True, check=True).stderr
    return {name: int(n) for name, n in re.findall(r"Function Name: (\S+).*?VGPRs Spill: (\d+)", report, re.S)}


@pytest.fixture(scope="module")
def rings():
    with ThreadPoolExecutor(5) as pool:
        return list(pool.map(spilled, ["keyswitch16_ring.hip:%d" % s for s in range(5)]))


def test_inner_products_over_transformed_digits_do_not_spill(rings):
    """Shared digits, of single rotations and of groups, for every kind of special primes."""
    for s, kernels in enumerate(rings):
        inner = {k: n for k, n in kernels.items() if "k_ks16_innerILi%dELb0E" % s in k}
        assert len(inner) == 6 and not any(inner.values()), (s, inner)


def test_forms_for_few_rotations_do_not_spill(rings):
    """A limb to a block, special limbs first, a wave to each digit; and the inverse column pass of up to three special primes (four take 128 registers for
    their residues alone, and some of the rest goes through scratch memory: 18, or 9 where the special limbs come first)."""
    for s, kernels in enumerate(rings):
        few = {k: n for k, n in kernels.items() if any(name + "ILi%d" % s in k for name in ("k_ks16_fcols_one", "k_ks16_specials", "k_ks16_inner_split"))}
        assert len(few) == 9 and not any(few.values()), (s, few)
        icols = {k: n for k, n in kernels.items() if "k_ks16_icolsILi%d" % s in k}
        assert len(icols) == 16, icols
        assert all(n <= (18 if "Li4E" in k.split("Arith")[1] else 0) for k, n in icols.items()), (s, icols)


def test_plane_splits_do_not_spill():
    """The splits of operands into planes, with and without the rescale, for every kind of digits, and the contraction."""
    kernels = spilled("accumulate_mfma.hip")
    assert len([k for k in kernels if "k_byte_planes_rescale" in k]) == 4 and not any(kernels.values()), kernels


def test_client_kernels_do_not_spill():
    """Encoding, encryption, decryption and decoding, on every ring."""
    kernels = {k: n for k, n in spilled("client16.hip").items() if "k_cl_" in k}
    assert len([k for k in kernels if "k_cl_icols_add" in k]) == 5 and not any(kernels.values()), kernels
