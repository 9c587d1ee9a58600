"""Ranges of the forward transform's values, of which only those that the first stage of a step adds to are reduced between steps
(fold_first).  The passes themselves, on an arithmetic whose numbers are bounds of the numbers that the device has.  Limits: 2^53 for doubles,
7.5 2^60 for the signed integers of primes just below 2^60."""
import hostdev

# Units of 2^50 > p: a product of y is within p / 2 + p |y| 2^-52 (the quotient: wp and the product are rounded), a folded value within p / 2 and the
# rounding of its quotient.  Units of 2^60: a product of x is within 1 + (1 + |x| / 8) 5 / 16, a folded value within 1/2 and 8 d / 2^60, d < 2^26.
PASSES = r"""
static double worst, folded, constant, slope;
struct Bounds {
    typedef double T;
    static double seen(double x) { if (x > worst) worst = x; return x; }
    T mid(T x) const { seen(x); return folded; }
    void ct(T &x, T &y, u64, u64) const { x = y = seen(x + constant + slope * seen(y)); }
};
static std::vector<double> shared(5000);
// every thread twice: in the second round it reads what all threads wrote in the first
template <int S>
static double cols(double start, bool fold) {
    typedef Ring<S> R;
    ulonglong2 tab[COL_TAB] = {};
    double end = 0;
    for (int t = 0; t < 512; t++) {
        double v[16];
        for (double &x : v) x = start;
        if (fold) fold_first(Bounds(), v);
        cols_fwd_tab<S>(Bounds(), v, tab, shared.data(), R::col(t & 255), R::grp(t & 255));
        if (t >= 256) for (double x : v) end = x > end ? x : end;
    }
    return end;
}
template <bool FROM_COLS>
static double rows(double start) {
    ulonglong2 tab[16] = {};
    double end = 0;
    for (int t = 0; t < 128; t++) {
        double v[16];
        for (double &x : v) x = start;
        row_fwd<FROM_COLS>(Bounds(), v, tab, tab, (u64 *)shared.data(), t >> 4 & 3, t & 15);
        if (t >= 64) for (double x : v) end = x > end ? x : end;
    }
    return end;
}
template <int S>
static void ring() {
    for (int wide = 0; wide < 2; wide++) {
        folded = 0.5 + (wide ? 0x1p-30 : 0x1p-40), constant = wide ? 1.3125 : 0.5, slope = wide ? 0.0390625 : 0.25, worst = 0;
        const double residue = cols<S>(wide ? 1.14 : 1.0, false), converted = wide ? residue : cols<S>(5.0, true);
        printf("%d %d %.4f %.4f ", S, wide, residue, converted);
        rows<true>(residue > converted ? residue : converted);
        printf("%.4f ", worst);
        worst = 0;
        rows<false>(1.0);
        printf("%.4f\n", worst);
    }
}
int main() { ring<0>(); ring<1>(); ring<2>(); ring<3>(); ring<4>(); }
"""


def test_values_stay_in_range_between_reductions(tmp_path):
    got = hostdev.run(tmp_path, PASSES)
    assert len(got) == 10
    for s, wide, residue, converted, whole, row in got:
        assert max(residue, converted, whole, row) < (6.9 if wide else 7.4), (s, wide, residue, converted, whole, row)  # below 7.5, and below 8
    # the first step of a column pass ends within 6.31 (the single step of the smallest ring), as the comment at fold_first says
    assert max(got[0][2:4]) < 6.31


def test_basis_conversion_starts_the_pass_in_range(tmp_path):
    """The sums of a conversion leave the reduction within p + 2^52, congruent to what went in; then the first eight of sixteen are folded."""
    hostdev.run(tmp_path, r"""
#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main() {
    for (u64 q : {(1ull << 50) - 27, (1ull << 49) + 1, (1ull << 45) - 55, (1ull << 36) - 5}) {
        PrimeConst pc = {};
        pc.q = q;
        pc.aux0 = (u64)__double_as_longlong(1.0 / (double)q);
        ArithFp ar;
        ar.init(pc);
        const int64_t big1 = (int64_t)1 << 53, big0 = (int64_t)1 << 52;
        for (int64_t a1 : {big1, big1 - 1, -big1, (int64_t)12345, (int64_t)0, -big1 + 77})
            for (int64_t a0 : {big0, big0 - 3, -big0, (int64_t)0, -(int64_t)1}) {
                const double r = ar.reduce25(a1, a0);
                CHECK(fabs(r) <= (double)q + 0x1p52 && r == rint(r));
                CHECK(((__int128)a1 * ((int64_t)1 << 25) + a0 - (int64_t)r) % (__int128)q == 0);
            }
        double v[16];
        for (int i = 0; i < 16; i++) v[i] = (i & 1 ? -1 : 1) * ((double)q + 0x1p52 - i);
        double w[16];
        memcpy(w, v, sizeof v);
        modup_fold(ar, w);
        for (int i = 0; i < 16; i++) {
            CHECK(((int64_t)w[i] - (int64_t)v[i]) % (int64_t)q == 0);
            CHECK(i < 8 ? fabs(w[i]) <= (double)q * (0.5 + 0x1p-30) + 1 : w[i] == v[i]);
        }
    }
    return 0;
}
""")
