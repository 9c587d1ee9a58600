"""The bounds that the signed arithmetic for primes just below 2^60 (ArithWide) rests on, for every prime it admits."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_09424_amd", "csrc")
Q60 = 1 << 60
LIMIT = 15 << 59  # the reduction adds 2^59 to a word before it shifts: beyond 7.5 2^60 that overflows

# For each ring: the largest admitted distance from 2^60, the primes of the transform that lie within it (the first 32 at most,
# as a context holds) and the multipliers among their 2N-th roots of unity, times 1 and 2^32, whose lower half exceeds 27 bits.
SCAN = r"""
#include <stdint.h>
#include <cstdio>
#include <initializer_list>
#include "hostmath.h"
int main() {
    u64 d = 1;
    while (hm_is_wide(((u64)1 << 60) - d)) d += 2;
    printf("%llu\n", (unsigned long long)(d - 2));
    for (int log_n = 12; log_n <= 16; log_n++) {
        const u64 two_n = (u64)2 << log_n;
        int primes = 0, longer = 0;
        for (u64 q = ((u64)1 << 60) - two_n + 1; hm_is_wide(q) && primes < 32; q -= two_n) {
            if (!hm_is_prime(q)) continue;
            primes++;
            u64 root = 0;
            for (u64 g = 2; !root; g++) {
                const u64 w = hm_powmod(g, (q - 1) / two_n, q);
                if (hm_powmod(w, two_n / 2, q) == q - 1) root = w;
            }
            u64 w = 1;
            for (u64 k = 0; k < two_n; k++, w = hm_mulmod(w, root, q))
                for (u64 m : {w, hm_mulmod(w, (u64)1 << 32, q)}) {
                    const int32_t lo = (int32_t)(u32)hm_wide_pack(m, q);
                    longer += lo > (1 << 27) || lo < -(1 << 27);
                }
        }
        printf("%d %d %d\n", log_n, primes, longer);
    }
}
"""


def test_bounds_of_the_wide_arithmetic(tmp_path):
    src, exe = tmp_path / "scan.cpp", tmp_path / "scan"
    src.write_text(SCAN)
    subprocess.run(["g++", "-O2", "-std=c++17", "-D__host__=", "-D__device__=", "-D__forceinline__=inline", "-I" + CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, check=True, timeout=300).stdout.split("\n")
    d = int(out[0])
    assert all(int(line.split()[1]) >= 8 and int(line.split()[2]) == 0 for line in out[1:6]), out

    def product(x):  # bounds of a product whose variable factor is within x: B 2^28 + A, B folded by 2^60 = d
        xh, xl, wh, wl = (x >> 32) + 1, 1 << 31, 1 << 31, 1 << 27
        a, b = (xh + xl) * wl, (xh + xl) * wh
        fold = (b >> 32) * d + d
        return -a - fold, a + fold + Q60

    # forward step: from the basis conversion (or a canonical residue, or a reduced word) four stages of x +- product
    x = Q60 + (1 << 57) + (1 << 27) * d
    for _ in range(4):
        lo, hi = product(x)
        x += max(-lo, hi)
    assert x < LIMIT, x / Q60
    # inverse steps of one to four stages on reduced words: the range of every element, the words that gs_fix folds among them
    word = (-(1 << 59) - 8 * d, (1 << 59) + 8 * d)
    for stages in range(1, 5):
        v = [word] * 16
        for k in range(stages - 1, -1, -1):
            if k == 0 and stages == 4:
                for i in (0, 1, 8, 9):
                    assert -LIMIT < v[i][0] and v[i][1] < LIMIT
                    v[i] = word
            for i in range(16):
                if not i & (8 >> k):
                    a, b = v[i], v[i + (8 >> k)]
                    v[i], diff = (a[0] + b[0], a[1] + b[1]), (a[0] - b[1], a[1] - b[0])
                    assert -LIMIT < diff[0] and diff[1] < LIMIT
                    v[i + (8 >> k)] = product(max(-diff[0], diff[1]))
            assert all(-LIMIT < lo and hi < LIMIT for lo, hi in v), (stages, k)
