// Arithmetic and register-level building blocks of the register transform (rings N = 2^12 .. 2^16), shared by the plain
// transform kernels, the fused key-switching kernels and the fused plaintext multiplication.
//
// A limb of N = 4096 * 2^S words, S = 0 .. 4, is viewed as 16 * 2^S rows of 256 (row-major).  The stages of the
// Cooley-Tukey network (Gentleman-Sande for the inverse) are cut S + 4 | 4 + 4: the column pass covers the stages whose
// butterflies span rows, the row pass those inside a row.  A step of up to four stages works on 16 values a thread holds in
// registers; the two steps of a pass exchange through LDS (a column pass at S = 0 is a single step).  A column tile is
// 256 / 2^S whole columns, 4096 words; a row tile is a number of whole rows; a limb has 2^S column tiles.
//
// Three arithmetic back ends with the same interface:
//   ArithFp   primes below 2^50: residues are exact integers held in doubles; a product
//             x*w mod p is  h = x*w; l = fma(x,w,-h); q = rint(x*(w/p)); r = fma(-q,p,h)+l
//             (exact: h - q*p and l are integers below 2^53).  Values stay within +-8p and
//             are brought back to |x| <= p/2 with x - rint(x/p)*p between inverse steps, half of them between
//             forward ones (fold_first).
//   ArithWide primes q = 2^60 - d, d < 2^26: signed 64-bit integers.  A multiplier w is stored as two centred residues w and
//             w 2^32 mod q, each split at 28 bits, so that x = xh 2^32 + xl (xl signed) times w is congruent to
//             B 2^28 + A with A, B two-term sums of 32 x 32 bit products; B's upper dword times 2^60 is folded with
//             2^60 = d.  Six multiply-adds and two more instructions where the Shoup product takes about twenty: a
//             32 x 32 + 64 bit multiply-add issues at the rate of an fp64 FMA on this chip (5.4 and 5.2 cycles of 2.4 GHz
//             per wave measured, held clock about 1.9 GHz), so what counts is the number of instructions -- eleven per
//             butterfly, against eight for ArithFp and about twenty-six for ArithInt.
//             Bounds, in units of 2^60 (the reduction takes |x| < 7.5): with |xl|, |wh| <= 2^31 and |wl| <= 2^27, A is
//             within (1 + |x| / 8) / 4, B's upper dword times d within (1 + |x| / 8) / 16, B's lower one times 2^28 in [0, 1): a
//             product of |x| < 7.5 is in (-0.61, 1.61).  (No power of a 2N-th root of unity, times 1 or 2^32, of an admitted
//             prime is one of the 2^27 multipliers below 2^59 whose lower half is longer.)  A forward step starts within
//             1.14 and grows to 2.49, 3.90, 5.37 and 6.89: no reduction in its four stages.  An inverse step starts within
//             0.51; sums double, a product restarts, so only the elements that are sums of three or four
//             stages would leave the range: they are folded before the last stage (gs_fix).
//   ArithInt  every other prime: 64-bit Shoup/Harvey lazy butterflies.
#pragma once
#include <type_traits>

#include "common.h"

// 32 x 32 + 64 bit multiply-adds; each is a single instruction (v_mad_i64_i32 / v_mad_u64_u32) as long as the compiler sees
// the widening of both factors next to the product, see keep_narrow.
__device__ __forceinline__ int64_t mul_i(int a, int b) { return (int64_t)a * b; }
__device__ __forceinline__ int64_t mad_i(int a, int b, int64_t c) { return (int64_t)a * b + c; }
__device__ __forceinline__ int64_t mad_uu(u32 a, u32 b, int64_t c) { return (int64_t)((u64)a * b + (u64)c); }
// a 2^k + c by one multiply-add: the factor is hidden from the compiler, which would make a shift and two adds of it
template <int K>
__device__ __forceinline__ int64_t mad_pow2(u32 a, int64_t c) {
    u32 f;
    asm("s_mov_b32 %0, %1" : "=s"(f) : "i"(1u << K));
    return mad_uu(a, f, c);
}
// To be called at the top of a loop on values that the loop does not change and multiplies by: the compiler would
// otherwise widen them once before the loop, which doubles their registers and leaves 64 x 64 bit products inside.
__device__ __forceinline__ void keep_narrow(u64 &x) { asm volatile("" : "+v"(x)); }

// A pointer that was itself read from memory: told to be global memory, so that its accesses are no generic ("flat") ones,
// which also occupy the LDS counters.
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) T *as_global(T *p) {
    return (__attribute__((address_space(1))) T *)p;
}

// Constant tables: scalar loads wherever the index is wave-uniform, whatever else the kernel stores.  (As ordinary memory
// they are vector loads in any loop that also stores, and the wait for one is a wait for every load issued before it.)
template <class T>
__device__ __forceinline__ const __attribute__((address_space(4))) T *as_const(const T *p) {
    return (const __attribute__((address_space(4))) T *)p;
}
__device__ __forceinline__ PrimeConst load_prime(const PrimeConst *pcs, int i) {
    static_assert(sizeof(PrimeConst) == 8 * sizeof(u64), "eight words");
    auto w = as_const((const u64 *)(pcs + i));
    return {w[0], w[1], w[2], w[3], w[4], w[5], w[6], w[7]};
}

// Word at a wave-uniform base plus a per-lane byte offset: the base stays in scalar registers.
__device__ __forceinline__ u64 ld_off(const u64 *base, u32 bytes) { return *(const u64 *)((const char *)base + bytes); }
__device__ __forceinline__ void st_off(u64 *base, u32 bytes, u64 x) { *(u64 *)((char *)base + bytes) = x; }

struct ArithInt {
    typedef u64 T;
    u64 q, two_q, ninv, ninv_s, qneg_inv;
    static __device__ __forceinline__ T from_bits(u64 x) { return x; }  // a workspace word
    __device__ __forceinline__ void init(const PrimeConst &pc) {
        q = pc.q;
        qneg_inv = pc.qneg_inv;
        two_q = 2 * pc.q;
        ninv = pc.n_inv;
        ninv_s = pc.n_inv_s;
    }
    __device__ __forceinline__ T load(u64 x) const { return x; }
    __device__ __forceinline__ T center(T x) const { return x; }
    __device__ __forceinline__ void ct(T &x, T &y, u64 w, u64 ws) const {  // in/out [0,4q)
        const T xs = csub(x, two_q);
        const T t = mul_shoup_lazy(y, w, ws, q);
        x = xs + t;
        y = xs - t + two_q;
    }
    __device__ __forceinline__ void gs(T &u, T &v, u64 w, u64 ws) const {  // in/out [0,2q)
        const T s = csub(u + v, two_q);
        v = mul_shoup_lazy(u - v + two_q, w, ws, q);
        u = s;
    }
    __device__ __forceinline__ T mid(T x) const { return x; }
    __device__ __forceinline__ u64 store_fwd(T x) const { return csub(csub(x, two_q), q); }
    __device__ __forceinline__ u64 store_inv(T x) const { return csub(x, q); }
    __device__ __forceinline__ u64 store_inv_scaled(T x) const { return mul_shoup(x, ninv, ninv_s, q); }
    // workspace words after a whole forward pass and an inverse row pass: the canonical residue; after a forward column pass: below 4 q
    __device__ __forceinline__ u64 store_ws_cols(T x) const { return x; }
    __device__ __forceinline__ u64 store_ws_fwd(T x) const { return store_fwd(x); }
    __device__ __forceinline__ u64 store_ws_inv(T x) const { return store_inv(x); }
    __device__ __forceinline__ void gs_fix(T *) const {}
};

struct ArithWide {
    typedef int64_t T;
    static __device__ __forceinline__ T from_bits(u64 x) { return (T)x; }
    int64_t q;
    int d, d4;
    u64 ninv, ninv_s;
    __device__ __forceinline__ void init(const PrimeConst &pc) {
        q = (int64_t)pc.q;
        d = (int)pc.aux0;
        d4 = 4 * d;
        ninv = pc.n_inv;
        ninv_s = pc.n_inv_s;
    }
    __device__ __forceinline__ T load(u64 x) const { return (T)x; }
    __device__ __forceinline__ T mul(T y, u64 w, u64 ws) const {
        const int xl = (int)(u32)y, xh = (int)(y >> 32) + (int)((u32)y >> 31);
        const int64_t b = mad_i(xh, (int)(ws >> 32), mul_i(xl, (int)(w >> 32)));
        const int64_t a = mad_i(xh, (int)(u32)ws, mul_i(xl, (int)(u32)w));
        return mad_pow2<28>((u32)b, mad_i((int)(b >> 32), d, a));
    }
    // |x| < 7.5 2^60 -> |result| <= 2^59 + 8 d
    __device__ __forceinline__ T mid(T x) const {
        const int hi = (int)(x >> 32), k = (hi + (1 << 27)) >> 28;
        const int h = __builtin_amdgcn_sbfe(hi, 0, 28);
        const T r = (T)(((u64)(u32)h << 32) | (u32)x);
        return mad_i(k, d, r);
    }
    __device__ __forceinline__ T center(T x) const { return mid(x); }
    // the residue in [-(q-1)/2, (q-1)/2]
    __device__ __forceinline__ T centred(T x) const {
        const T half = q >> 1;
        T r = mid(x);
        r = r > half ? r - q : r;
        return r < -half ? r + q : r;
    }
    __device__ __forceinline__ u64 canon(T x) const {
        const T r = mid(x);
        return (u64)(r < 0 ? r + q : r);
    }
    __device__ __forceinline__ void ct(T &x, T &y, u64 w, u64 ws) const {
        const T t = mul(y, w, ws);
        y = x - t;
        x = x + t;
    }
    __device__ __forceinline__ void gs(T &u, T &v, u64 w, u64 ws) const {
        const T s = u + v;
        v = mul(u - v, w, ws);
        u = s;
    }
    __device__ __forceinline__ void gs_fix(T *v) const {
        v[0] = mid(v[0]);
        v[1] = mid(v[1]);
        v[8] = mid(v[8]);
        v[9] = mid(v[9]);
    }
    __device__ __forceinline__ u64 store_fwd(T x) const { return canon(x); }
    __device__ __forceinline__ u64 store_inv(T x) const { return canon(x); }
    __device__ __forceinline__ u64 store_inv_scaled(T x) const { return canon(mul(x, ninv, ninv_s)); }
    // workspace word after a forward pass: the centred value as high * 2^30 + low, two int32 halves
    __device__ __forceinline__ u64 store_ws_fwd(T x) const {
        const T r = mid(x) + (1 << 29);
        const u32 hi = (u32)(u64)(r >> 30), lo = ((u32)r & 0x3fffffffu) - (1u << 29);
        return ((u64)hi << 32) | lo;
    }
    __device__ __forceinline__ u64 store_ws_cols(T x) const { return (u64)x; }
    __device__ __forceinline__ u64 store_ws_inv(T x) const { return (u64)mid(x); }
};

struct ArithFp {
    typedef double T;
    double p, pinv, ninv, ninv_p;
    static __device__ __forceinline__ T from_bits(u64 x) { return __longlong_as_double((long long)x); }
    __device__ __forceinline__ void init(const PrimeConst &pc) {
        p = (double)pc.q;
        pinv = __longlong_as_double((long long)pc.aux0);
        ninv = (double)pc.n_inv;
        ninv_p = __longlong_as_double((long long)pc.aux1);
    }
    // An integer in [0, 2^52) is the mantissa of that integer plus 2^52: two instructions each way, where the conversions take
    // four and seven.
    static __device__ __forceinline__ T from_residue(u64 x) { return __longlong_as_double((long long)(x | 0x4330000000000000ull)) - 0x1p52; }
    static __device__ __forceinline__ u64 to_residue(T x) { return (u64)__double_as_longlong(x + 0x1p52) & 0xfffffffffffffull; }
    __device__ __forceinline__ T load(u64 x) const { return from_residue(x); }
    __device__ __forceinline__ T mid(T x) const { return fma(-rint(x * pinv), p, x); }  // -> |x| <= p/2
    __device__ __forceinline__ T center(T x) const { return mid(x); }
    __device__ __forceinline__ T mulmod(T y, T w, T wp) const {  // |y| < 2^53 -> |result| < 2.5p, exact integer
        const double h = y * w;
        const double l = fma(y, w, -h);
        const double q = rint(y * wp);
        return fma(-q, p, h) + l;
    }
    // x*k mod p for a multiplier without a precomputed k/p: |x| <= p/2, 0 <= k < p -> |result| < 0.7p, exact integer
    __device__ __forceinline__ T mulmod_np(T x, T k) const {
        const double h = x * k;
        const double l = fma(x, k, -h);
        const double q = rint(h * pinv);
        return fma(-q, p, h) + l;
    }
    __device__ __forceinline__ void ct(T &x, T &y, u64 w, u64 ws) const {
        const T t = mulmod(y, __longlong_as_double((long long)w), __longlong_as_double((long long)ws));
        y = x - t;
        x = x + t;
    }
    __device__ __forceinline__ void gs(T &u, T &v, u64 w, u64 ws) const {
        const T s = u + v;
        v = mulmod(u - v, __longlong_as_double((long long)w), __longlong_as_double((long long)ws));
        u = s;
    }
    __device__ __forceinline__ u64 canon(T x) const {
        T r = mid(x);
        r = r < 0.0 ? r + p : r;
        return to_residue(r);
    }
    __device__ __forceinline__ u64 store_fwd(T x) const { return canon(x); }
    __device__ __forceinline__ u64 store_inv(T x) const { return canon(x); }
    __device__ __forceinline__ u64 store_inv_scaled(T x) const { return canon(mulmod(x, ninv, ninv_p)); }
    // workspace words: the bits of the double, |x| <= p/2 (after a forward column pass: below 8 p)
    __device__ __forceinline__ u64 store_ws_fwd(T x) const { return (u64)__double_as_longlong(mid(x)); }
    __device__ __forceinline__ u64 store_ws_cols(T x) const { return (u64)__double_as_longlong(x); }
    __device__ __forceinline__ u64 store_ws_inv(T x) const { return store_ws_fwd(x); }
    __device__ __forceinline__ void gs_fix(T *) const {}
    // a number congruent to a1 2^25 + a0 mod p for |a1| <= 2^53, |a0| <= 2^52: within p + 2^52
    __device__ __forceinline__ T reduce25(int64_t a1, int64_t a0) const {
        const double x = fma((double)(int)(a1 >> 32), 4294967296.0, (double)(u32)a1) * 33554432.0;
        const double y = fma((double)(int)(a0 >> 32), 4294967296.0, (double)(u32)a0);
        return fma(-rint(x * pinv), p, x) + y;
    }
    // the same for |a1|, |a0| < 2^60: their dwords are taken apart, |result| <= p + 2^32
    __device__ __forceinline__ T reduce25_long(int64_t a1, int64_t a0) const {
        const double x = (double)(int)(a1 >> 32) * 0x1p57;
        const double m = fma((double)(int)(a0 >> 32), 4294967296.0, (double)(u32)a1 * 33554432.0);  // a multiple of 2^25 below 2^61
        const double r = fma(-rint(x * pinv), p, x);
        return fma(-rint(m * pinv), p, m) + r + (double)(u32)a0;
    }
};

// Four Cooley-Tukey stages on 16 elements whose local index i is the 4 index bits of the step
// (bit 3 = largest distance).  tw/tws: the prime's forward table and its companion.
template <class A>
__device__ __forceinline__ void ct4(const A &ar, typename A::T *v, const u64 *tw, const u64 *tws, u32 mbase) {
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const int d = 8 >> k;
#pragma unroll
        for (int g = 0; g < (1 << k); g++) {
            const u64 w = tw[(mbase << k) + g], ws = tws[(mbase << k) + g];
#pragma unroll
            for (int o = 0; o < d; o++) {
                const int i0 = g * 2 * d + o;
                ar.ct(v[i0], v[i0 + d], w, ws);
            }
        }
    }
}
// ct4 with the step's 15 twiddles (value, companion) already at hand: entry (1 << k) - 1 + g serves local stage k,
// butterfly group g.  TAB is anything indexable that yields .x (value) and .y (companion) as 64-bit words -- a table
// in LDS shared by the threads of a row, or a per-thread array in registers -- so that a kernel that runs the same
// step on several limbs in a row fetches the twiddles once.
template <class A, class TAB>
__device__ __forceinline__ void ct4_tab(const A &ar, typename A::T *v, const TAB &tab) {
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const int d = 8 >> k;
#pragma unroll
        for (int g = 0; g < (1 << k); g++) {
            const u64 w = tab[(1 << k) - 1 + g].x, ws = tab[(1 << k) - 1 + g].y;
#pragma unroll
            for (int o = 0; o < d; o++) {
                const int i0 = g * 2 * d + o;
                ar.ct(v[i0], v[i0 + d], w, ws);
            }
        }
    }
}
// The tables' last 15/16 serve the second steps of the row pass, 15 entries for each thread of a wave's four rows.  They lie in the
// order in which waves read them: entry e (ct4_tab's order) of lane l of the four rows 4 t .. 4 t + 3 at N / 16 + 960 t +
// row_twiddle_pos(e, l).  In the order of the network a load of the last stage's eight entries touched a line for every two lanes: 680 lines
// a wave and table against the 120 that it reads, nearly as many as all operands of an inner product.
ENSI_HD u32 row_twiddle_pos(u32 e, u32 l) { return e < 14 ? (e >> 1) * 128 + l * 2 + (e & 1) : 896 + l; }
// place of entry k >= N / 16 of a table in the network's order, rows of 256
ENSI_HD u32 row_twiddle_place(u32 k, u32 n) {
    u32 stage = 0;
    while (k >> stage >= n / 8) stage++;
    const u32 rem = k - (n / 16 << stage), g = rem & ((1u << stage) - 1), rj = rem >> stage, r = rj >> 4;
    return n / 16 + (r >> 2) * 960 + row_twiddle_pos((1u << stage) - 1 + g, (r & 3) * 16 + (rj & 15));
}
typedef u64 word_pair __attribute__((vector_size(16)));
// The 15 twiddles of a thread in the second step of the row pass, in ct4_tab's order.
struct TwRegs {
    ulonglong2 t[15];
    __device__ __forceinline__ const ulonglong2 &operator[](int i) const { return t[i]; }
    __device__ __forceinline__ void keep() {
#pragma unroll
        for (int i = 0; i < 15; i++) {
            u64 x = t[i].x, y = t[i].y;
            keep_narrow(x);
            keep_narrow(y);
            t[i] = make_ulonglong2(x, y);
        }
    }
    // those of thread j of row r, second step, of a ring of n words
    __device__ __forceinline__ void load(const u64 *tw, const u64 *tws, u32 n, u32 r, u32 j) {
        const u32 at = n / 16 + (r >> 2) * 960, lane = (r & 3) * 16 + j;
#pragma unroll
        for (int e = 0; e < 14; e += 2) {
            const word_pair a = *(const word_pair *)(tw + at + row_twiddle_pos(e, lane)), b = *(const word_pair *)(tws + at + row_twiddle_pos(e, lane));
            t[e] = make_ulonglong2(a[0], b[0]);
            t[e + 1] = make_ulonglong2(a[1], b[1]);
        }
        t[14] = make_ulonglong2(tw[at + row_twiddle_pos(14, lane)], tws[at + row_twiddle_pos(14, lane)]);
    }
};

// The inverse of ct4 up to the factor 16 (inverse table).
template <class A>
__device__ __forceinline__ void gs4(const A &ar, typename A::T *v, const u64 *tw, const u64 *tws, u32 mbase) {
#pragma unroll
    for (int k = 3; k >= 0; k--) {
        const int d = 8 >> k;
        if (k == 0) ar.gs_fix(v);
#pragma unroll
        for (int g = 0; g < (1 << k); g++) {
            const u64 w = tw[(mbase << k) + g], ws = tws[(mbase << k) + g];
#pragma unroll
            for (int o = 0; o < d; o++) {
                const int i0 = g * 2 * d + o;
                ar.gs(v[i0], v[i0 + d], w, ws);
            }
        }
    }
}
// gs4 with the step's twiddles at hand (see ct4_tab).
template <class A, class TAB>
__device__ __forceinline__ void gs4_tab(const A &ar, typename A::T *v, const TAB &tab) {
#pragma unroll
    for (int k = 3; k >= 0; k--) {
        const int d = 8 >> k;
        if (k == 0) ar.gs_fix(v);
#pragma unroll
        for (int g = 0; g < (1 << k); g++) {
            const u64 w = tab[(1 << k) - 1 + g].x, ws = tab[(1 << k) - 1 + g].y;
#pragma unroll
            for (int o = 0; o < d; o++) {
                const int i0 = g * 2 * d + o;
                ar.gs(v[i0], v[i0 + d], w, ws);
            }
        }
    }
}
// Thread (rho, j) of a row tile puts entry j < 15 of row rho's step table (base index mbase_row, which depends on the row
// only) into tab[rho * 16 + j]; the caller orders that before the first use.
__device__ __forceinline__ void row_table_to_lds(ulonglong2 *tab, const u64 *tw, const u64 *tws, u32 mbase_row, int rho, int j) {
    if (j < 15) {
        const int k = 31 - __clz(j + 1), g = j + 1 - (1 << k);
        const u32 idx = (mbase_row << k) + g;
        tab[rho * 16 + j] = make_ulonglong2(tw[idx], tws[idx]);
    }
}

// ---- pass bodies on registers ------------------------------------------------------
template <int S>
struct Ring {
    static constexpr int LOGN = 12 + S;
    static constexpr int N = 4096 << S;
    static constexpr int ROWS = 16 << S;
    static constexpr int TILES = 1 << S;        // column tiles, and 16-row tiles, of a limb
    static constexpr int LOGC = 8 - S;          // a column tile is 2^LOGC columns
    static constexpr int COLS = 1 << LOGC;
    // thread tid of a column tile: column tid % COLS, row group tid / COLS
    static __device__ __forceinline__ int col(int tid) { return tid & (COLS - 1); }
    static __device__ __forceinline__ int grp(int tid) { return tid >> LOGC; }
    // the row of value i on the side of the first forward / last inverse step (on the other side: 16 jj + i)
    static __device__ __forceinline__ int row(int jj, int i) { return ((i >> (4 - S)) << 4) + (jj << (4 - S)) + (i & ((1 << (4 - S)) - 1)); }
};

// Brings the first eight of a forward step's values back to their range.  In the step's first stage value i + 8 is multiplied, which leaves
// it small whatever it was, and added to and subtracted from value i: reducing the ones that are added to is enough.  In units of p (ArithFp,
// primes just below 2^50; a product of y is within 1/2 + |y| / 4, its quotient's rounding): the first step of a column pass starts within 1 (or, folded, within 1/2 and 5 after
// the basis conversion) and ends within 6.31, the ones after it start within 1/2 and 7.4 and end within 7.4 again, below the 8 = 2^53
// that a double holds.  (ArithWide, units of 2^60: 1/2 and 6.9, ending within 6.5, below 7.5.)  Reducing all sixteen took 3 instructions a word
// more per pass.
template <class A>
__device__ __forceinline__ void fold_first(const A &ar, typename A::T *v) {
#pragma unroll
    for (int i = 0; i < 8; i++) v[i] = ar.mid(v[i]);
}

// The first ST stages of a forward step and the last ST of an inverse one, all over the same 15 twiddles.
template <int ST, class A, class TAB>
__device__ __forceinline__ void ct_first_tab(const A &ar, typename A::T *v, const TAB &tab) {
#pragma unroll
    for (int k = 0; k < ST; k++) {
        const int d = 8 >> k;
#pragma unroll
        for (int g = 0; g < (1 << k); g++) {
            const u64 w = tab[(1 << k) - 1 + g].x, ws = tab[(1 << k) - 1 + g].y;
#pragma unroll
            for (int o = 0; o < d; o++) ar.ct(v[g * 2 * d + o], v[g * 2 * d + o + d], w, ws);
        }
    }
}
// TIGHT: the twiddles of a stage are read when it begins, not all at once (they would take 60 registers)
template <int ST, class A, class TAB, bool TIGHT = false>
__device__ __forceinline__ void gs_last_tab(const A &ar, typename A::T *v, const TAB &tab) {
#pragma unroll
    for (int k = ST - 1; k >= 0; k--) {
        const int d = 8 >> k;
        if (TIGHT) __builtin_amdgcn_sched_barrier(0);
        if (k == 0 && ST == 4) ar.gs_fix(v);
#pragma unroll
        for (int g = 0; g < (1 << k); g++) {
            const u64 w = tab[(1 << k) - 1 + g].x, ws = tab[(1 << k) - 1 + g].y;
#pragma unroll
            for (int o = 0; o < d; o++) ar.gs(v[g * 2 * d + o], v[g * 2 * d + o + d], w, ws);
        }
    }
}
// The 15 twiddles of base index 1 where they lie in memory (the same for every thread).
struct TwFirst {
    const u64 *tw, *tws;
    struct Pair {
        u64 x, y;
    };
    __device__ __forceinline__ Pair operator[](int i) const { return {as_const(tw)[i + 1], as_const(tws)[i + 1]}; }
};

// Column pass of a 256-thread block on one column tile; lds holds 4096 words.
//   forward: on entry v[i] = row Ring::row(jj, i) of the thread's column, on exit v[i] = row 16 jj + i.
//   inverse: on entry v[i] = row 16 jj + i (|v| <= p/2 for ArithFp and ArithWide, [0,2q) for ArithInt), on exit
//            v[i] = row Ring::row(jj, i), not yet multiplied by 1/N.
// Neither synchronises after its last LDS read: the caller must, before the tile is reused.
template <int S, class A>
__device__ __forceinline__ void cols_fwd_regs(const A &ar, typename A::T *v, const u64 *tw, const u64 *tws, void *lds, int c, int jj) {
    typedef Ring<S> R;
    if (S > 0) {
        typename A::T *l = (typename A::T *)lds;
        ct_first_tab<S>(ar, v, TwFirst{tw, tws});
#pragma unroll
        for (int i = 0; i < 16; i++) l[R::row(jj, i) * R::COLS + c] = v[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 16; i++) v[i] = l[(16 * jj + i) * R::COLS + c];
        fold_first(ar, v);
    }
    ct4(ar, v, tw, tws, (1u << S) + jj);
}
template <int S, class A>
__device__ __forceinline__ void cols_inv_regs(const A &ar, typename A::T *v, const u64 *tw, const u64 *tws, void *lds, int c, int jj) {
    typedef Ring<S> R;
    gs4(ar, v, tw, tws, (1u << S) + jj);
    if (S > 0) {
        typename A::T *l = (typename A::T *)lds;
#pragma unroll
        for (int i = 0; i < 16; i++) l[(16 * jj + i) * R::COLS + c] = ar.mid(v[i]);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 16; i++) v[i] = l[R::row(jj, i) * R::COLS + c];
        gs_last_tab<S>(ar, v, TwFirst{tw, tws});
    }
}

// The same passes with the twiddles of the tile in LDS, for a block that walks several limbs: entry e < 15 of slot 0 serves
// the first step, of slot 1 + jj the second step of row group jj (ct4_tab's order; 16 entries a slot).  Every thread has at
// most one entry to fetch (col_tab_index, col_tab_fetch), so the table of the next limb is requested while the current one
// is transformed, put into LDS before the pass's barrier and complete for everybody after it: no pass waits for a
// twiddle.
#define COL_TAB 272
template <int S>
__device__ __forceinline__ int col_tab_index(int tid, u32 *idx) {  // returns the entry's place, -1 for none
    const int slot = tid / 15, e = tid - slot * 15;
    if (slot > (1 << S)) return -1;
    const int k = 31 - __clz(e + 1), g = e + 1 - (1 << k);
    *idx = ((slot == 0 ? 1u : (1u << S) + slot - 1) << k) + g;
    return slot * 16 + e;
}
template <int S, class A>
__device__ __forceinline__ void cols_fwd_tab(const A &ar, typename A::T *v, const ulonglong2 *tab, void *lds, int c, int jj) {
    typedef Ring<S> R;
    if (S > 0) {
        typename A::T *l = (typename A::T *)lds;
        ct_first_tab<S>(ar, v, tab);
#pragma unroll
        for (int i = 0; i < 16; i++) l[R::row(jj, i) * R::COLS + c] = v[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 16; i++) v[i] = l[(16 * jj + i) * R::COLS + c];
        fold_first(ar, v);
    } else {
        __syncthreads();
    }
    ct4_tab(ar, v, tab + 16 * (1 + jj));
}
template <int S, class A>
__device__ __forceinline__ void cols_inv_tab(const A &ar, typename A::T *v, const ulonglong2 *tab, void *lds, int c, int jj) {
    typedef Ring<S> R;
    gs_last_tab<4, A, const ulonglong2 *, true>(ar, v, tab + 16 * (1 + jj));
    if (S > 0) {
        typename A::T *l = (typename A::T *)lds;
#pragma unroll
        for (int i = 0; i < 16; i++) l[(16 * jj + i) * R::COLS + c] = ar.mid(v[i]);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 16; i++) v[i] = l[R::row(jj, i) * R::COLS + c];
        gs_last_tab<S, A, const ulonglong2 *, true>(ar, v, tab);
    } else {
        __syncthreads();
    }
}

// Row pass.  The 16 threads of a row sit in one wave, so a wave runs four whole rows by itself and its exchanges need no
// barrier, only the order of its own LDS accesses.  Thread (rho = lane / 16, j = lane % 16); l: the wave's ROW_LDS words of
// LDS (one pad word per 16: the strided and the contiguous pattern are both free of conflicts); rows: rows of the limb.
//   forward: on entry v[i] = element j + 16 i of row rho, on exit v[i] = element 16 j + i.
//   inverse: on entry v[i] = element 16 j + i, on exit v[i] = element j + 16 i.
#define ROW_LDS (1024 + 64)
// Register order of a wave's four rows in the key switch: where value i of a lane lies among their 1024 words.  A lane's even value and
// the odd one behind it are neighbours: loads of 16 bytes a lane.
__device__ __forceinline__ u32 reg_pos(int i, int lane) { return (u32)((i >> 1) * 128 + lane * 2 + (i & 1)); }
__device__ __forceinline__ int rpad(int p) { return p + (p >> 4); }
// Orders a wave's LDS writes before the reads of its other lanes that follow.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// tab1: the row's first-step twiddles (row_table_to_lds), tab2: the thread's second-step twiddles, in ct4_tab's order
// FROM_COLS: the values are as a forward column pass left them (store_ws_cols), else canonical residues
template <bool FROM_COLS, class A, class TAB1, class TAB2>
__device__ __forceinline__ void row_fwd(const A &ar, typename A::T *v, const TAB1 &tab1, const TAB2 &tab2, u64 *lds, int rho, int j) {
    typename A::T *l = (typename A::T *)lds;
    if (FROM_COLS) fold_first(ar, v);
    ct4_tab(ar, v, tab1);
#pragma unroll
    for (int i = 0; i < 16; i++) l[rpad(rho * 256 + j + 16 * i)] = v[i];
    wave_lds_fence();
#pragma unroll
    for (int i = 0; i < 16; i++) v[i] = l[rpad(rho * 256 + 16 * j + i)];
    fold_first(ar, v);
    ct4_tab(ar, v, tab2);
    wave_lds_fence();
}
template <class A, class TAB1, class TAB2>
__device__ __forceinline__ void row_inv(const A &ar, typename A::T *v, const TAB1 &tab1, const TAB2 &tab2, u64 *lds, int rho, int j) {
    typename A::T *l = (typename A::T *)lds;
    gs4_tab(ar, v, tab2);
#pragma unroll
    for (int i = 0; i < 16; i++) l[rpad(rho * 256 + 16 * j + i)] = ar.mid(v[i]);
    wave_lds_fence();
#pragma unroll
    for (int i = 0; i < 16; i++) v[i] = l[rpad(rho * 256 + j + 16 * i)];
    gs4_tab(ar, v, tab1);
    wave_lds_fence();
}

__device__ __forceinline__ u32 brev8(u32 x) { return __brev(x) >> 24; }

// phi_g on transform-domain positions.  Position k holds the evaluation at psi^(2 brev(k) + 1) and phi_g(d)(psi^x) = d(psi^(x g)):
// output row r reads one source row, within which position p reads brev8(g brev8(p) + carry mod 256), where the carry
// comes from the row's part of the exponent.  Four rows 4t .. 4t + 3 read four rows 4t' .. 4t' + 3.
template <int S>
struct RowMap {
    static constexpr int LOGR = 4 + S;
    static constexpr u32 ROWS = 1u << LOGR;
    static __device__ __forceinline__ u32 exponent(u32 row) { return 2 * (__brev(row) >> (32 - LOGR)) + 1; }
    static __device__ __forceinline__ u32 row(u32 exp) { return __brev((exp & (2 * ROWS - 1)) >> 1) >> (32 - LOGR); }
    static __device__ __forceinline__ u32 source(u32 r, u32 g) { return row(g * exponent(r)); }
    static __device__ __forceinline__ u32 carry(u32 r, u32 g) { return g * exponent(r) >> (LOGR + 1) & 255; }
};

// Calls f with the ring's S as a compile-time constant (12 <= log_n <= 16).
template <class F>
inline void ring_dispatch(int log_n, F f) {
    switch (log_n) {
        case 12: f(std::integral_constant<int, 0>{}); break;
        case 13: f(std::integral_constant<int, 1>{}); break;
        case 14: f(std::integral_constant<int, 2>{}); break;
        case 15: f(std::integral_constant<int, 3>{}); break;
        default: f(std::integral_constant<int, 4>{}); break;
    }
}
