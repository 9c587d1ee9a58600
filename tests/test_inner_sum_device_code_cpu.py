"""The sums of up to eight products that the inner product of the key switch reduces once: the device's own steps, at the ends of their range."""
import pytest

import hostdev
from paper_2509_09424_amd import binding

SUMS = r"""
#define CHECK(x) do { if (!(x)) { printf("line %d: %s (p %llu, %d products)\n", __LINE__, #x, (unsigned long long)q, n); return 1; } } while (0)
static u64 bits(double d) { return (u64)__double_as_longlong(d); }
int main() {
    for (u64 q : {(1ull << 50) - 27, (1ull << 49) + 1, (1ull << 45) - 55, (1ull << 36) - 5, (1ull << 20) + 7}) {
        PrimeConst pc = {};
        pc.q = q;
        pc.aux0 = bits(1.0 / (double)q);
        ArithFp ar;
        ar.init(pc);
        const double e = (double)(q / 2);
        for (int n : {1, 4, 8})
            for (int signs = 0; signs < 4; signs++)
                for (int odd : {0, 1, 12345})
                    for (double c0 : {e, -e, 0.0}) {
                        Inner<ArithFp>::Sum s;
                        __int128 want = (int64_t)c0;
                        for (int i = 0; i < n; i++) {
                            const double x = (signs & 1 ? -1 : 1) * (e - odd), k = (signs & 2 ? -1 : 1) * (e - 2 * odd * (i % 2));
                            want += (__int128)(int64_t)x * (int64_t)k;
                            s.mac(bits(x), bits(k));
                            CHECK(s.h >= 0x1p102 && s.h < 0x1p103 && fabs(s.l) <= 0x1p52);
                        }
                        // nothing is lost: what the two words hold is the sum itself
                        CHECK((__int128)((s.h - 0x1.8p102) * 0x1p-50) * ((__int128)1 << 50) + (int64_t)s.l == want - (int64_t)c0);
                        s.add(bits(c0));
                        const double got = s.reduced(ar);
                        CHECK(got == rint(got) && fabs(got) <= (double)q * (0.5 + 0x1p-30) + 1);
                        CHECK((want - (int64_t)got) % (__int128)q == 0);
                    }
    }
    for (u64 q : {(1ull << 61) - 1, (1ull << 61) - 31, (1ull << 55) + 9}) {  // any odd modulus does for the reduction
        PrimeConst pc = {};
        pc.q = q;
        u64 inv = 1;
        for (int i = 0; i < 6; i++) inv *= 2 - q * inv;
        pc.qneg_inv = 0 - inv;
        ArithInt ar;
        ar.init(pc);
        for (int n : {1, 4, 8})
            for (u64 x : {q - 1, q / 2, (u64)1, (u64)0}) {
                Inner<ArithInt>::Sum s;
                for (int i = 0; i < n; i++) s.mac(x, q - 1 - i);
                unsigned __int128 left = 0;
                for (int i = 0; i < n; i++) left = (left + (unsigned __int128)x * (q - 1 - i) % q) % q;
                const u64 got = s.reduced(ar);
                unsigned __int128 back = got;  // got 2^64 is the sum
                for (int i = 0; i < 64; i++) back = back * 2 % q;
                CHECK(got < q && back == left);
            }
    }
    return 0;
}
"""


def test_sums_at_the_ends_of_their_range(tmp_path):
    hostdev.run(tmp_path, SUMS)


def test_no_more_digits_than_the_sums_hold():
    with pytest.raises(binding.EnsiError, match="code -1"):
        binding.Context(12, 50, 9, 60, 1, 1, 40, seed=1)
