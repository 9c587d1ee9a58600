// Rotation (paper, Preliminaries: Rot) for the rings N = 2^12 .. 2^16 with ciphertext primes below 2^50:
// automorphism plus hybrid key switching in three kernels (four where more than RAISE_ONE_MAX rotations share one raised
// ciphertext) that keep every intermediate in the layout and number format of the transform passes around it.
//
//   k_ks16_fcols   ModUp fused into the forward column pass.  A block holds the inner factors
//                  y_a = c1_a (Q_j/q_a)^-1 mod q_a of one digit on one column tile in registers and walks the
//                  limbs of the extended basis: it forms  sum_a y_a (Q_j/q_a) mod t  (or takes the limb inside its
//                  own digit), runs the column pass on it and writes it.  Further blocks do the same for P * c0, so
//                  that phi_g(c0) can be added in the transform domain (ModDown divides it by P again, exactly)
//   k_ks16_frows   forward row pass of the raised digits and of P * c0, where more than RAISE_ONE_MAX rotations read them
//   k_ks16_inner   inner product with the key + P * c0, automorphism (a permutation of transform-domain positions that maps
//                  rows onto rows) of the two sums, inverse row pass.  A raised ciphertext that fewer rotations read is taken after its column
//                  pass and the row passes of its digits are run here: the transformed digits never reach memory
//   k_ks16_icols   inverse column pass fused with ModDown.  A block brings the K special limbs of one column tile
//                  to centred residues y_k = [u (P/p_k)^-1]_{p_k}, held in registers, and then walks the
//                  ciphertext limbs:  u P^-1 - sum_k y_k p_k^-1  mod q_i
//
// Few rotations, which do not fill the chip, take forms with more and shorter blocks: k_ks16_fcols_one (a limb to a block), k_ks16_specials
// (the special limbs of the accumulators first) and k_ks16_inner_split (a wave to each digit); where the lines lie is said at the launchers.
//
// What bounds them: a row or column pass costs 40 to 60 instructions per word, the memory system about as much, so
// neither can be wasted.  Holding y (fcols) and y_k (icols) in registers while the block walks the limbs is what
// removed the re-reads: with a block per limb each word of y was fetched through L2 once per target limb and the
// kernels waited on those loads, whatever their arithmetic cost.
//
// Number formats between the kernels (workspaces only, never visible outside the library), by
// the prime's kind:
//   PRIME_FP    doubles (exact integers, |x| <= p/2; after a forward column pass below 8 p); key: the same
//   PRIME_WIDE  signed 64-bit integers, |x| <= q/2 + 8 (2^60 - q) (after a forward column pass below 7.5 2^60); transformed digits and the key as two
//               int32 halves high * 2^30 + low, so that the inner product is multiply-adds of 32-bit words
//   PRIME_INT   canonical 64-bit residues (after a forward column pass below 4 q); key: Montgomery residues
// Transformed digits and the key are stored in the order a wave holds them in the row pass ("register order"): within
// the four rows of a wave, value i of lane (rho, j) -- position 16 j + i of row rho -- at reg_pos(i, lane), so that reading
// them needs no exchange and is contiguous, two values to a load.  The key of element g lies at the positions its words meet before the automorphism:
// phi_g^-1 of it is stored.
// All results that leave the last kernel are canonical residues and equal, word for word, what the unfused sequence
// (ModUp, transform, inner product, inverse transform, ModDown, + phi_g(c0)) gives.
#pragma once
#include "common.h"
#include "ntt16_core.h"

#define KS_THREADS 256

__device__ __forceinline__ int ks_ext_prime(int e, int l1, int L) { return e < l1 ? e : L + (e - l1); }
__device__ __forceinline__ double as_f64(u64 x) { return __longlong_as_double((long long)x); }
__device__ __forceinline__ u64 as_u64(double x) { return (u64)__double_as_longlong(x); }

__device__ __forceinline__ RotDesc load_desc(const RotDesc *desc, int i) {
    static_assert(sizeof(RotDesc) == 6 * sizeof(u64), "six words");
    auto w = as_const((const u64 *)(desc + i));
    RotDesc d;
    d.c0 = (const u64 *)w[0];
    d.digits = (const u64 *)w[1];
    d.key = (const u64 *)w[2];
    d.out = (u64 *)w[3];
    d.g = (u32)w[4];
    d.g_inv = (u32)(w[4] >> 32);
    d.accumulate = (u32)w[5];
    return d;
}

// ------------------------------------------------------------------ ModUp + forward column pass
// Basis conversion of values h .. h+7 of a column: sum_a y_a h_a over the 25-bit halves of y against split h and
// h 2^25 is a1 2^b + a0 (b = 25 or 30: where the halves of h meet); four multiply-adds per source, one reduction
// per word afterwards (a modular product per source in fp64 took twice the instructions).
template <int Y>
__device__ __forceinline__ void modup_sums(int64_t *a0, int64_t *a1, const u64 *hat, u64 (*y)[Y], int ns, int h) {
#pragma unroll
    for (int a = 0; a < ENSI_MAX_ALPHA; a++) {
        if (a == 0 || a < ns) {  // (ns >= 1)
            const u64 w = as_const(hat)[2 * a], w25 = as_const(hat)[2 * a + 1];
#pragma unroll
            for (int i = 0; i < 8; i++) {
                const int yl = (int)(u32)y[a][h + i], yh = (int)(y[a][h + i] >> 32);
                a0[i] = mad_i(yh, (int)(u32)w25, a ? mad_i(yl, (int)(u32)w, a0[i]) : mul_i(yl, (int)(u32)w));
                a1[i] = mad_i(yh, (int)(w25 >> 32), a ? mad_i(yl, (int)(w >> 32), a1[i]) : mul_i(yl, (int)(w >> 32)));
            }
        }
    }
}

template <int Y>
__device__ __forceinline__ void modup_half(const ArithFp &ar, double *v, const u64 *hat, const u64 *, u64 (*y)[Y], int ns, const PrimeConst &, int h) {
    int64_t a0[8], a1[8];
    modup_sums(a0, a1, hat, y, ns, h);
#pragma unroll
    for (int i = 0; i < 8; i++) v[i] = ar.reduce25(a1[i], a0[i]);
}
// |a0|, |a1| <= 2^57 leave the value within 1.14 q, as a forward step may start
template <int Y>
__device__ __forceinline__ void modup_half(const ArithWide &ar, int64_t *v, const u64 *hat, const u64 *, u64 (*y)[Y], int ns, const PrimeConst &, int h) {
    int64_t a0[8], a1[8];
    modup_sums(a0, a1, hat, y, ns, h);
#pragma unroll
    for (int i = 0; i < 8; i++) v[i] = mad_pow2<30>((u32)a1[i] & 0x3fffffffu, mad_i((int)(a1[i] >> 30), ar.d, a0[i]));
}
template <int Y>
__device__ __forceinline__ void modup_half(const ArithInt &, u64 *v, const u64 *, const u64 *hat_mont, u64 (*y)[Y], int ns, const PrimeConst &pc, int h) {
#pragma unroll
    for (int i = 0; i < 8; i++) {
        acc128 acc = {0, 0};
#pragma unroll
        for (int a = 0; a < ENSI_MAX_ALPHA; a++)
            if (a < ns) mac128(acc, (y[a][h + i] >> 32 << 25) | (u32)y[a][h + i], as_const(hat_mont)[a]);
        v[i] = mont_reduce(acc, pc.q, pc.qneg_inv);
    }
}
// what the first stage of the column pass asks of the sums
__device__ __forceinline__ void modup_fold(const ArithFp &ar, double *v) { fold_first(ar, v); }
template <class A>
__device__ __forceinline__ void modup_fold(const A &, typename A::T *) {}
template <class A>
__device__ __forceinline__ void modup_to(const A &ar, typename A::T *v, const u64 *hat, const u64 *hat_mont, u64 (*y)[16], int ns, const PrimeConst &pc) {
#pragma unroll
    for (int h = 0; h < 16; h += 8) modup_half(ar, v + h, hat, hat_mont, y, ns, pc, h);
    modup_fold(ar, v);
}
// y_a as two halves of 25 bits, from a word of c1
__device__ __forceinline__ u64 modup_factor(u64 x, u64 inv, u64 inv_s, u64 q) {
    const u64 t = mul_shoup(x, inv, inv_s, q);
    return (t >> 25) << 32 | (t & 0x1ffffffu);
}

// LDS of a block that walks limbs, one barrier per pass.  A thread past the barrier of pass t may write the tile of pass
// t + 1 while another still reads the tile of pass t: two tiles in turn.  The table of pass t + 1 is written before the
// barrier of pass t, when another thread may still be reading the table of pass t - 1: three tables in turn.
struct ColLds {
    ulonglong2 tab[3][COL_TAB];
    u64 tile[2][4096];
};

// grid (TILES, beta * ceil(ext / per) + ceil(l1 / per), n_ct): a block takes `per` targets of one digit, or `per` limbs of
// P * c0.  dig: [n_ct][beta*ext + l1][N], row R < beta*ext is limb R % ext of raised digit R / ext.
// W: the arithmetic of the special primes (one kind for all of them).
template <int S, class W>
__global__ __launch_bounds__(KS_THREADS, 2) void k_ks16_fcols(Ks16Const kc, const PrimeConst *pcs, const u64 *tw_all, const u64 *ct_base,
                                                              size_t ct_stride, int limb_stride, u64 *dig, int per) {
    typedef Ring<S> R;
    constexpr size_t N = R::N;
    __shared__ ColLds sh;
    const int tid = threadIdx.x, c = R::col(tid), jj = R::grp(tid);
    const int l1 = kc.l1, ext = l1 + kc.K, chunks = (ext + per - 1) / per;
    const u64 *c0 = ct_base + (size_t)blockIdx.z * ct_stride + (size_t)blockIdx.x * R::COLS;
    u64 *out_ct = dig + (size_t)blockIdx.z * (kc.beta * ext + l1) * N + (size_t)blockIdx.x * R::COLS;
    const u32 off_in = (R::row(jj, 0) * 256 + c) * 8, off_out = (16 * jj * 256 + c) * 8;  // of value 0; value i adds the same for all threads
    u32 tidx = 0;
    const int tplace = col_tab_index<S>(tid, &tidx);
    ulonglong2 tnext;
    auto fetch_tab = [&](int prime) {
        const u64 *tw = tw_all + (size_t)prime * 4 * N;
        tnext = make_ulonglong2(tw[tidx], tw[N + tidx]);
    };
    auto put_tab = [&](int buf) {
        if (tplace >= 0) sh.tab[buf][tplace] = tnext;
    };
    if ((int)blockIdx.y < kc.beta * chunks) {
        const u64 *c1 = c0 + (size_t)limb_stride * N;
        const int j = blockIdx.y / chunks, e0 = (blockIdx.y - j * chunks) * per, e1 = min(ext, e0 + per);
        const int first = j * kc.alpha, ns = kc.n_src[j];
        fetch_tab(ks_ext_prime(e0, l1, kc.L));
        u64 y[ENSI_MAX_ALPHA][16] = {};
#pragma unroll
        for (int a = 0; a < ENSI_MAX_ALPHA; a++) {
            if (a < ns) {
                const u64 q = load_prime(pcs, first + a).q, inv = as_const(kc.inv)[first + a], inv_s = as_const(kc.inv_s)[first + a];
                const u64 *src = c1 + (size_t)(first + a) * N;
#pragma unroll
                for (int i = 0; i < 16; i++) y[a][i] = ld_off(src + R::row(0, i) * 256, off_in);
#pragma unroll
                for (int i = 0; i < 16; i++) y[a][i] = modup_factor(y[a][i], inv, inv_s, q);
            }
        }
        put_tab(0);
        __syncthreads();
        int tcur = 0;
#pragma unroll 1
        for (int e = e0; e < e1; e++) {
#pragma unroll
            for (int a = 0; a < ENSI_MAX_ALPHA; a++)
#pragma unroll
                for (int i = 0; i < 16; i++) keep_narrow(y[a][i]);
            const int prime = ks_ext_prime(e, l1, kc.L);
            const PrimeConst pc = load_prime(pcs, prime);
            const u64 *hat = kc.hat_sp + ((size_t)j * ext + e) * kc.alpha * 2;
            u64 *out = out_ct + ((size_t)j * ext + e) * N, *l = sh.tile[e & 1];
            const int tnxt = tcur == 2 ? 0 : tcur + 1;
            const ulonglong2 *tb = sh.tab[tcur];
            tcur = tnxt;
            if (e + 1 < e1) fetch_tab(ks_ext_prime(e + 1, l1, kc.L));
            if (e < l1) {
                ArithFp ar;
                ar.init(pc);
                double v[16];
                if (e >= first && e < first + ns) {
#pragma unroll
                    for (int i = 0; i < 16; i++) v[i] = ar.load(ld_off(c1 + (size_t)e * N + R::row(0, i) * 256, off_in));
                } else {
                    modup_to(ar, v, hat, (const u64 *)nullptr, y, ns, pc);
                }
                put_tab(tnxt);
                cols_fwd_tab<S>(ar, v, tb, l, c, jj);
#pragma unroll
                for (int i = 0; i < 16; i++) st_off(out + i * 256, off_out, ar.store_ws_cols(v[i]));
            } else {
                W ar;
                ar.init(pc);
                typename W::T v[16];
                modup_to(ar, v, hat, kc.hat_mont + ((size_t)j * ext + e) * kc.alpha, y, ns, pc);
                put_tab(tnxt);
                cols_fwd_tab<S>(ar, v, tb, l, c, jj);
#pragma unroll
                for (int i = 0; i < 16; i++) st_off(out + i * 256, off_out, ar.store_ws_cols(v[i]));
            }
        }
    } else {
        const int i0 = (blockIdx.y - kc.beta * chunks) * per, i1 = min(l1, i0 + per);
        fetch_tab(i0);
        u64 nv[16];
#pragma unroll
        for (int i = 0; i < 16; i++) nv[i] = ld_off(c0 + (size_t)i0 * N + R::row(0, i) * 256, off_in);
        put_tab(0);
        __syncthreads();
        int tcur = 0;
#pragma unroll 1
        for (int limb = i0; limb < i1; limb++) {
            ArithFp ar;
            ar.init(load_prime(pcs, limb));
            const double pm = as_const(kc.pmod_fp)[2 * limb], pm_p = as_const(kc.pmod_fp)[2 * limb + 1];
            double v[16];
#pragma unroll
            for (int i = 0; i < 16; i++) v[i] = ar.mulmod(ar.load(nv[i]), pm, pm_p);
            if (limb + 1 < i1) {
                fetch_tab(limb + 1);
#pragma unroll
                for (int i = 0; i < 16; i++) nv[i] = ld_off(c0 + (size_t)(limb + 1) * N + R::row(0, i) * 256, off_in);
            }
            const int tnxt = tcur == 2 ? 0 : tcur + 1;
            put_tab(tnxt);
            cols_fwd_tab<S>(ar, v, sh.tab[tcur], sh.tile[limb & 1], c, jj);
            tcur = tnxt;
            u64 *out = out_ct + (size_t)(kc.beta * ext + limb) * N;
#pragma unroll
            for (int i = 0; i < 16; i++) st_off(out + i * 256, off_out, ar.store_ws_cols(v[i]));
        }
    }
}

// The same for few ciphertexts, a limb to a block: the factors y_a are formed for the one target, half a column at a time, so that four
// blocks fit a CU where a walk over limbs leaves room for two.  grid (TILES, beta * ext + l1, n_ct)
struct ColLdsOne {
    ulonglong2 tab[COL_TAB];
    u64 tile[4096];
};
template <int S, class A>
__device__ __forceinline__ void fcols_one_body(const Ks16Const &kc, const PrimeConst *pcs, const PrimeConst &pc, const u64 *c, u64 *out, int row, u32 off_in, u32 off_out,
                                               ColLdsOne &sh, int col, int jj) {
    typedef Ring<S> R;
    constexpr size_t N = R::N;
    const int l1 = kc.l1, ext = l1 + kc.K, j = row / ext, first = j * kc.alpha, ns = kc.n_src[j];
    A ar;
    ar.init(pc);
    typename A::T v[16];
    const u64 *hat = kc.hat_sp + (size_t)row * kc.alpha * 2, *hat_mont = kc.hat_mont + (size_t)row * kc.alpha;
#pragma unroll
    for (int h = 0; h < 16; h += 8) {
        u64 y[ENSI_MAX_ALPHA][8];
#pragma unroll
        for (int a = 0; a < ENSI_MAX_ALPHA; a++) {
            if (a < ns) {
#pragma unroll
                for (int i = 0; i < 8; i++) y[a][i] = ld_off(c + (size_t)(first + a) * N + R::row(0, h + i) * 256, off_in);
            }
        }
#pragma unroll
        for (int a = 0; a < ENSI_MAX_ALPHA; a++) {
            if (a < ns) {
                const u64 q = load_prime(pcs, first + a).q, inv = as_const(kc.inv)[first + a], inv_s = as_const(kc.inv_s)[first + a];
#pragma unroll
                for (int i = 0; i < 8; i++) y[a][i] = modup_factor(y[a][i], inv, inv_s, q);
            }
        }
        modup_half(ar, v + h, hat, hat_mont, y, ns, pc, 0);
    }
    modup_fold(ar, v);
    cols_fwd_tab<S>(ar, v, sh.tab, sh.tile, col, jj);
#pragma unroll
    for (int i = 0; i < 16; i++) st_off(out + i * 256, off_out, ar.store_ws_cols(v[i]));
}
template <int S, class W>
__global__ __launch_bounds__(KS_THREADS, 4) void k_ks16_fcols_one(Ks16Const kc, const PrimeConst *pcs, const u64 *tw_all, const u64 *ct_base, size_t ct_stride,
                                                                  int limb_stride, u64 *dig) {
    typedef Ring<S> R;
    constexpr size_t N = R::N;
    __shared__ ColLdsOne sh;
    const int tid = threadIdx.x, c = R::col(tid), jj = R::grp(tid), row = blockIdx.y;
    const int l1 = kc.l1, ext = l1 + kc.K, rows = kc.beta * ext, limb = row < rows ? row % ext : row - rows, prime = row < rows ? ks_ext_prime(limb, l1, kc.L) : limb;
    const u64 *c0 = ct_base + (size_t)blockIdx.z * ct_stride + (size_t)blockIdx.x * R::COLS, *c1 = c0 + (size_t)limb_stride * N;
    u64 *out = dig + ((size_t)blockIdx.z * (rows + l1) + row) * N + (size_t)blockIdx.x * R::COLS;
    const u32 off_in = (R::row(jj, 0) * 256 + c) * 8, off_out = (16 * jj * 256 + c) * 8;
    const u64 *tw = tw_all + (size_t)prime * 4 * N;
    u32 tidx = 0;
    const int tplace = col_tab_index<S>(tid, &tidx);
    if (tplace >= 0) sh.tab[tplace] = make_ulonglong2(tw[tidx], tw[N + tidx]);
    const PrimeConst pc = load_prime(pcs, prime);
    const int first = row < rows ? row / ext * kc.alpha : 0;
    if (row >= rows || (limb >= first && limb < first + kc.n_src[row / ext])) {  // P * c0, or the digit's own limb
        const bool is_c0 = row >= rows;
        const double pm = as_const(kc.pmod_fp)[2 * limb], pm_p = as_const(kc.pmod_fp)[2 * limb + 1];
        ArithFp ar;
        ar.init(pc);
        double v[16];
#pragma unroll
        for (int i = 0; i < 16; i++) v[i] = ar.load(ld_off((is_c0 ? c0 : c1) + (size_t)limb * N + R::row(0, i) * 256, off_in));
        if (is_c0) {
#pragma unroll
            for (int i = 0; i < 16; i++) v[i] = ar.mulmod(v[i], pm, pm_p);
        }
        __syncthreads();
        cols_fwd_tab<S>(ar, v, sh.tab, sh.tile, c, jj);
#pragma unroll
        for (int i = 0; i < 16; i++) st_off(out + i * 256, off_out, ar.store_ws_cols(v[i]));
        return;
    }
    __syncthreads();
    if (limb < l1) fcols_one_body<S, ArithFp>(kc, pcs, pc, c1, out, row, off_in, off_out, sh, c, jj);
    else fcols_one_body<S, W>(kc, pcs, pc, c1, out, row, off_in, off_out, sh, c, jj);
}

// ------------------------------------------------------------------ forward row pass (in place)
// A wave runs its four rows of one limb for up to KS_FROWS_GROUP ciphertexts: the twiddles of the rows -- more bytes than
// the rows themselves -- are fetched once (first step: LDS, second step: registers), and the next ciphertext's rows are
// requested before the current ones are transformed.  grid (4 TILES * (beta*ext + l1) * ceil(n_ct / KS_FROWS_GROUP)).
#define KS_FROWS_GROUP 8
template <int S, class A>
__device__ __forceinline__ void frows_body(u64 *g, size_t ct_stride, int n_here, const u64 *tw, const PrimeConst &pc, u64 *lds, ulonglong2 *tw1,
                                           int r0) {
    A ar;
    ar.init(pc);
    const int lane = threadIdx.x, rho = lane >> 4, j = lane & 15;
    const u32 base = Ring<S>::ROWS + r0 + rho;
    const u64 *tws = tw + Ring<S>::N;
    row_table_to_lds(tw1, tw, tws, base, rho, j);
    TwRegs tw2;
    tw2.load(tw, tws, Ring<S>::N, r0 + rho, j);
    const ulonglong2 *tab = tw1 + rho * 16;
    typename A::T v[16], nv[16];
    {
        const typename A::T *gt = (const typename A::T *)g;
#pragma unroll
        for (int i = 0; i < 16; i++) nv[i] = gt[rho * 256 + j + 16 * i];
    }
    wave_lds_fence();
#pragma unroll 1
    for (int c = 0; c < n_here; c++) {
        tw2.keep();
#pragma unroll
        for (int i = 0; i < 16; i++) v[i] = nv[i];
        if (c + 1 < n_here) {
            const typename A::T *gt = (const typename A::T *)(g + (size_t)(c + 1) * ct_stride);
#pragma unroll
            for (int i = 0; i < 16; i++) nv[i] = gt[rho * 256 + j + 16 * i];
        }
        row_fwd<true>(ar, v, tab, tw2, lds, rho, j);
        u64 *go = g + (size_t)c * ct_stride;
#pragma unroll
        for (int i = 0; i < 16; i += 2) *(word_pair *)(go + reg_pos(i, lane)) = word_pair{ar.store_ws_fwd(v[i]), ar.store_ws_fwd(v[i + 1])};
    }
}

template <int S, class W>
__global__ __launch_bounds__(64, 2) void k_ks16_frows(Ks16Const kc, const PrimeConst *pcs, const u64 *tw_all, u64 *dig, int n_ct) {
    typedef Ring<S> R;
    __shared__ u64 lds[ROW_LDS];
    __shared__ ulonglong2 tw1[4 * 16];
    // The ciphertext group runs fastest: blocks that share a part of the twiddle table (same limb, same rows) are
    // launched together and fetch it from memory once per XCD.
    const int n_grp = (n_ct + KS_FROWS_GROUP - 1) / KS_FROWS_GROUP;
    const int grp = blockIdx.x % n_grp, tile = (blockIdx.x / n_grp) % (4 * R::TILES), row = blockIdx.x / (n_grp * 4 * R::TILES);
    const int l1 = kc.l1, ext = l1 + kc.K, n_rows = kc.beta * ext + l1;
    const int prime = row < kc.beta * ext ? ks_ext_prime(row % ext, l1, kc.L) : row - kc.beta * ext;
    const PrimeConst pc = load_prime(pcs, prime);
    const u64 *tw = tw_all + (size_t)prime * 4 * R::N;
    const int r0 = tile * 4, ct0 = grp * KS_FROWS_GROUP;
    const int n_here = min(KS_FROWS_GROUP, n_ct - ct0);
    const size_t ct_stride = (size_t)n_rows * R::N;
    u64 *g = dig + ((size_t)ct0 * n_rows + row) * R::N + (size_t)r0 * 256;
    if (prime < kc.L) frows_body<S, ArithFp>(g, ct_stride, n_here, tw, pc, lds, tw1, r0);
    else frows_body<S, W>(g, ct_stride, n_here, tw, pc, lds, tw1, r0);
}

// ---------------------------------------- automorphism + key inner product + inverse row pass
// Sums of products of transformed digit words x with key words k, both as 64-bit words in their stored formats.  mac: onto a sum
// that is reduced after each product.  Sum: the products of a whole inner product (at most 8 digits) are added first and
// reduced once; it holds two or three words where the other holds one.
template <class A>
struct Inner;
template <>
struct Inner<ArithFp> {
    static __device__ __forceinline__ void mac(const ArithFp &ar, double &s, u64 x, u64 k) { s += ar.mulmod_np(as_f64(x), as_f64(k)); }
    // h - 3 2^101 is the sum of the products rounded to multiples of 2^50, l what that rounding left: |x|, |k| <= p/2 < 2^49, so
    // eight products stay below 2^101 and h between 2^102 and 2^103; what one addition leaves is within 2^49, an integer that the second
    // multiply-add returns exactly, and |l| stays below 2^53 with P * c0 and the reduced h added.  Four instructions a product
    // instead of seven.
    struct Sum {
        double h = 0x1.8p102, l = 0.0;
        __device__ __forceinline__ void mac(u64 x, u64 k) {
            const double n = fma(as_f64(x), as_f64(k), h);
            l += fma(as_f64(x), as_f64(k), h - n);
            h = n;
        }
        __device__ __forceinline__ void add(u64 x) { l += as_f64(x); }
        __device__ __forceinline__ double reduced(const ArithFp &ar) const {
            const double t = h - 0x1.8p102;
            return ar.mid(fma(-rint(t * ar.pinv), ar.p, t) + l);
        }
    };
    static __device__ __forceinline__ double plus(const ArithFp &ar, double a, double b) { return ar.mid(a + b); }
    // up to nine terms, to be folded afterwards
    static __device__ __forceinline__ double plus_lazy(const ArithFp &, double a, double b) { return a + b; }
    static __device__ __forceinline__ void add(double &s, u64 x) { s += as_f64(x); }
    static __device__ __forceinline__ void fold(const ArithFp &ar, double &s) { s = ar.mid(s); }
    static __device__ __forceinline__ void settle(const ArithFp &ar, double &s) { s = ar.mid(s); }  // a sum of mac
};
// x = xh 2^30 + xl, k = kh 2^30 + kl: xh kh 2^60 is taken apart into dwords and folded by 2^60 = d, 2^62 = 4 d, like the
// middle sum m 2^30.  Every half is at most 2^29 (a little more for the high ones): within 6 q before the last fold, 6.6 q for the
// sum of eight products.
template <>
struct Inner<ArithWide> {
    static __device__ __forceinline__ int64_t folded(const ArithWide &ar, int64_t h, int64_t m, int64_t l) {
        m = mad_i((int)(h >> 32), ar.d4, m);
        l = mad_uu((u32)h, (u32)ar.d, l);
        return ar.mid(mad_pow2<30>((u32)m, mad_i((int)(m >> 32), ar.d4, l)));
    }
    static __device__ __forceinline__ void mac(const ArithWide &ar, int64_t &s, u64 x, u64 k) {
        const int xl = (int)(u32)x, xh = (int)(x >> 32), kl = (int)(u32)k, kh = (int)(k >> 32);
        s = folded(ar, mul_i(xh, kh), mad_i(xh, kl, mul_i(xl, kh)), mad_i(xl, kl, s));
    }
    struct Sum {
        int64_t h = 0, m = 0, l = 0;
        __device__ __forceinline__ void mac(u64 x, u64 k) {
            const int xl = (int)(u32)x, xh = (int)(x >> 32), kl = (int)(u32)k, kh = (int)(k >> 32);
            h = mad_i(xh, kh, h);
            m = mad_i(xh, kl, mad_i(xl, kh, m));
            l = mad_i(xl, kl, l);
        }
        __device__ __forceinline__ void add(u64) {}
        __device__ __forceinline__ int64_t reduced(const ArithWide &ar) const { return folded(ar, h, m, l); }
    };
    static __device__ __forceinline__ int64_t plus(const ArithWide &ar, int64_t a, int64_t b) { return ar.mid(a + b); }
    static __device__ __forceinline__ int64_t plus_lazy(const ArithWide &, int64_t a, int64_t b) { return a + b; }
    static __device__ __forceinline__ void add(int64_t &, u64) {}
    static __device__ __forceinline__ void fold(const ArithWide &ar, int64_t &s) { s = ar.mid(s); }
    static __device__ __forceinline__ void settle(const ArithWide &, int64_t &) {}
};
template <>
struct Inner<ArithInt> {
    static __device__ __forceinline__ void mac(const ArithInt &ar, u64 &s, u64 x, u64 k) { s = add_mod(s, mont_mul(x, k, ar.q, ar.qneg_inv), ar.q); }
    // eight Montgomery products of residues below 2^61 and the sum of their high words fit 128 bits: one reduction
    struct Sum {
        acc128 s = {0, 0};
        __device__ __forceinline__ void mac(u64 x, u64 k) { mac128(s, x, k); }
        __device__ __forceinline__ void add(u64) {}
        __device__ __forceinline__ u64 reduced(const ArithInt &ar) const { return mont_reduce(s, ar.q, ar.qneg_inv); }
    };
    static __device__ __forceinline__ u64 plus(const ArithInt &ar, u64 a, u64 b) { return add_mod(a, b, ar.q); }
    static __device__ __forceinline__ u64 plus_lazy(const ArithInt &ar, u64 a, u64 b) { return add_mod(a, b, ar.q); }
    static __device__ __forceinline__ void add(u64 &, u64) {}
    static __device__ __forceinline__ void fold(const ArithInt &, u64 &) {}
    static __device__ __forceinline__ void settle(const ArithInt &, u64 &) {}
};

// Four rows of one limb of both accumulators, by one wave, and their inverse row passes.  Digits and keys are multiplied where they
// lie -- keys are stored at the source positions of their element (k_ks16_key_format) -- and the automorphism permutes the
// two sums, not the beta + 1 polynomials they are made of.
//   GROUP = false: one rotation; the wave takes source rows 4 tile .. 4 tile + 3 and writes the rows they map to.
//   GROUP = true:  `members` rotations whose sums are added: the wave takes output rows 4 tile .. 4 tile + 3.
// RAW (not GROUP): the digits have only been through their column pass; their row passes are run here.
//
// What bounds the form that reads transformed digits (one rotation of the 2^16 ring at 16 + 4 limbs: 13 us, 14.6 before): the 21 MB of results
// that it writes (a quarter of the time by themselves) and the words that come through a CU's L1, 106 KB a tile and rotation.  Those
// come 16 bytes to a lane (8 bytes a lane reach 18 TB/s from L2, 16 bytes 34), keys once for the rotations of a block (those that
// use one key are neighbours), twiddles in the order they are read in.  An accumulator to each wave, four waves to a SIMD, takes 18 %
// longer, as every digit is then read twice; two and three waves to a SIMD are within 4 %.
// Rotations of a block, one to a wave: four where there are many, which share the lines of a key in the L1 of their CU; one where there are few, as a block
// of waves that have no rotation keeps its LDS, and one of waves that have leaves other CUs empty.  Inner products against one wave and
// four, over special primes of all kinds (geometric means, the kernel before blocks of four = 1): fills of one ciphertext on 2^15 and 2^16 1.07, 1.11, of five
// 0.95, 1.18, of 17 1.00, 1.01, of 40 0.955, 0.926; 3 to 15 rotations of a ciphertext 0.92 to 1.04, 0.94 to 1.05, 30 0.984, 0.990, 60 0.966, 0.910; on 2^12 to 2^14 five
// 0.91, 0.95, 30 0.941, 0.953, 60 0.933, 0.924.  The row-pass form never gains by a second wave (nine rotations 0.99, 1.03, 64 0.995, 0.998).
#define INNER_WAVES 4
#define INNER_WAVES_MIN 32  // rotations, or groups, from which a block has INNER_WAVES
struct InnerLds {  // of a wave
    u64 row[ROW_LDS];
    ulonglong2 tw1[4 * 16];
};
// Values of a row that one pass over the digits adds up, and waves to a SIMD, by the arithmetic of the special primes: what its registers
// allow without spilling.
template <bool GROUP, class W>
struct InnerShape {
    static constexpr int VALUES = std::is_same<W, ArithInt>::value ? 2 : 4, PER_SIMD = !GROUP && std::is_same<W, ArithWide>::value ? 3 : 2;
};
template <int S, bool RAW, bool GROUP, int C, class A>
__device__ __forceinline__ void inner_body(const Ks16Const &kc, const RotDesc *desc, const PrimeConst &pc, const u64 *tw_all, u64 *u, int prime, int e,
                                           int members, u32 grp, u32 tile, u64 *lds, ulonglong2 *tw1) {
    typedef Ring<S> R;
    typedef RowMap<S> M;
    typedef Inner<A> I;
    typedef typename A::T T;
    constexpr size_t N = R::N;
    const int lane = threadIdx.x & 63, rho = lane >> 4, j = lane & 15;
    const int l1 = kc.l1, ext = l1 + kc.K, beta = kc.beta;
    const size_t kstride = (size_t)(kc.L + kc.K) * N;  // words between b_j and a_j, and half the distance between digits
    const u64 *tw = tw_all + (size_t)prime * 4 * N;
    const ulonglong2 *tab = tw1 + rho * 16;
    A ar;
    ar.init(pc);
    T a0[16], a1[16];
    u32 r = tile * 4 + rho, g = 1, carry = 0;
    // Moves a sum from the positions that the element g reads (carry: of this row) to those that the next rotation's element reads,
    // or, with 1 and 0, to the output's own order.  The rotations of a group add to one pair of sums in this way; a
    // second pair in the output's order took 14 to 58 registers more than there are (fills of 384 and 768 ciphertexts, 15 limbs: 48.7
    // and 79.1 ms of inner products with it, 46.0 and 75.0 so).
    auto move = [&](T *a, u32 to_g_inv, u32 to_carry) {
        T *l = (T *)lds;
        // value i of lane j, position p = 16 j + i with brev8(p) = brev4(j) + 16 brev4(i), is at brev8(h (brev8(p) - to_carry) + carry)
        const u32 h = g * to_g_inv, first = h * ((__brev((u32)j) >> 28) - to_carry) + carry;
#pragma unroll
        for (int i = 0; i < 16; i++) l[rpad(rho * 256 + 16 * j + i)] = a[i];
        wave_lds_fence();
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const u32 brev4_i = (i & 1) * 8 + (i & 2) * 2 + (i & 4) / 2 + (i & 8) / 8;
            a[i] = l[rpad(rho * 256 + brev8(first + h * (16 * brev4_i)))];
        }
        wave_lds_fence();
    };
#pragma unroll 1
    for (int mem = 0; mem < (GROUP ? members : 1); mem++) {
        const RotDesc d = load_desc(desc, grp * members + mem);
        const u32 rs = GROUP ? M::source(r, d.g) : r;
        if (!GROUP) r = M::row(d.g_inv * M::exponent(rs));
        const u32 to_carry = M::carry(r, d.g);
        // byte offsets of value 0 from the wave's tile of digits and keys
        const u32 reg_off = ((GROUP ? (rs >> 2) * 1024 : 0) + reg_pos(0, (GROUP ? rs & 3 : rho) * 16 + j)) * 8, row_off = (rho * 256 + j) * 8;
        const u64 *src = d.digits + (size_t)e * N + (GROUP ? 0 : tile * 1024), *key = d.key + (size_t)prime * N + (GROUP ? 0 : tile * 1024);
        auto ld = [](const u64 *base, u32 off) { return *(decltype(as_global(base)))((decltype(as_global((const char *)base)))as_global(base) + off); };
        const bool with_c0 = e < l1;  // P * c0 follows the digits
        auto ld_pair = [](const u64 *base, u32 off) { return *(__attribute__((address_space(1))) const word_pair *)((decltype(as_global((const char *)base)))as_global(base) + off); };
        if (RAW) {
            TwRegs tw2;
            row_table_to_lds(tw1, tw, tw + N, R::ROWS + rs, rho, j);
            tw2.load(tw, tw + N, N, rs, j);
            u64 nv[16];
#pragma unroll
            for (int i = 0; i < 16; i++) {
                a0[i] = a1[i] = 0;
                nv[i] = ld(src + 16 * i, row_off);
            }
            wave_lds_fence();
            const int nd = with_c0 ? beta + 1 : beta;
#pragma unroll 1
            for (int jd = 0; jd < nd; jd++) {
                tw2.keep();
                T v[16];
#pragma unroll
                for (int i = 0; i < 16; i++) v[i] = A::from_bits(nv[i]);
                if (jd + 1 < nd) {
                    src += (size_t)ext * N;
#pragma unroll
                    for (int i = 0; i < 16; i++) nv[i] = ld(src + 16 * i, row_off);
                }
                row_fwd<true>(ar, v, tab, tw2, lds, rho, j);
                if (jd < beta) {
#pragma unroll
                    for (int h = 0; h < 16; h += 8) {
                        u64 k0[8], k1[8];
#pragma unroll
                        for (int i = 0; i < 8; i += 2) {
                            const word_pair p0 = ld_pair(key + reg_pos(h + i, 0), reg_off), p1 = ld_pair(key + kstride + reg_pos(h + i, 0), reg_off);
                            k0[i] = p0[0], k0[i + 1] = p0[1];
                            k1[i] = p1[0], k1[i + 1] = p1[1];
                        }
#pragma unroll
                        for (int i = 0; i < 8; i++) {
                            const u64 x = ar.store_ws_fwd(v[h + i]);
                            I::mac(ar, a0[h + i], x, k0[i]);
                            I::mac(ar, a1[h + i], x, k1[i]);
                        }
                    }
                    key += 2 * kstride;
                } else {
#pragma unroll
                    for (int i = 0; i < 16; i++) I::add(a0[i], ar.store_ws_fwd(v[i]));
                }
            }
        } else {
            // C values at a time over all digits (so that only theirs are sums of several words), the operands of the next product
            // requested before the current one is formed.
            u64 x[C], k0[C], k1[C];
            auto fetch = [&](const u64 *s, const u64 *k, bool keys) {
                auto get = [&](u64 *to, const u64 *from) {
#pragma unroll
                    for (int i = 0; i < C; i += 2) {
                        const word_pair p = ld_pair(from + reg_pos(i, 0), reg_off);
                        to[i] = p[0];
                        to[i + 1] = p[1];
                    }
                };
                get(x, s);
                if (keys) {
                    get(k0, k);
                    get(k1, k + kstride);
                }
            };
            fetch(src, key, true);
            if (GROUP && mem > 0) {
                move(a0, d.g_inv, to_carry);
                move(a1, d.g_inv, to_carry);
            }
#pragma unroll
            for (int i0 = 0; i0 < 16; i0 += C) {
                typename I::Sum s0[C], s1[C];
                const u64 *s = src + reg_pos(i0, 0), *k = key + reg_pos(i0, 0);
                auto product = [&](auto &&next) {
                    u64 cx[C], c0[C], c1[C];
#pragma unroll
                    for (int i = 0; i < C; i++) {
                        cx[i] = x[i];
                        c0[i] = k0[i];
                        c1[i] = k1[i];
                    }
                    next();
#pragma unroll
                    for (int i = 0; i < C; i++) {
                        s0[i].mac(cx[i], c0[i]);
                        s1[i].mac(cx[i], c1[i]);
                    }
                };
                auto fetch_next = [&] {
                    if (i0 + C < 16) fetch(src + reg_pos(i0 + C, 0), key + reg_pos(i0 + C, 0), true);
                };
#pragma unroll 2
                for (int jd = 1; jd < beta; jd++) {
                    s += (size_t)ext * N;
                    k += 2 * kstride;
                    product([&] { fetch(s, k, true); });
                }
                if (with_c0) {
                    product([&] { fetch(s + (size_t)ext * N, nullptr, false); });
                    u64 cx[C];
#pragma unroll
                    for (int i = 0; i < C; i++) cx[i] = x[i];
                    fetch_next();
#pragma unroll
                    for (int i = 0; i < C; i++) s0[i].add(cx[i]);
                } else {
                    product(fetch_next);
                }
#pragma unroll
                for (int i = 0; i < C; i++) {
                    T t0 = s0[i].reduced(ar), t1 = s1[i].reduced(ar);
                    asm volatile("" : "+v"(t0), "+v"(t1));  // here, not where they are used: until then each would be two or three words
                    a0[i0 + i] = GROUP && mem > 0 ? I::plus(ar, a0[i0 + i], t0) : t0;
                    a1[i0 + i] = GROUP && mem > 0 ? I::plus(ar, a1[i0 + i], t1) : t1;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (RAW) {
#pragma unroll
            for (int i = 0; i < 16; i++) {
                I::settle(ar, a0[i]);
                I::settle(ar, a1[i]);
            }
        }
        g = d.g;
        carry = to_carry;
        if (!GROUP || mem + 1 == members) {
            move(a0, 1, 0);  // the automorphism within the rows
            move(a1, 1, 0);
        }
    }
    // inverse row pass of both sums: its twiddles are fetched once
    tw += 2 * N;
    row_table_to_lds(tw1, tw, tw + N, R::ROWS + r, rho, j);
    TwRegs twi;
    twi.load(tw, tw + N, N, r, j);
    wave_lds_fence();
    u64 *uo = u + ((size_t)grp * 2 * ext + e) * N + (size_t)r * 256 + j;
#pragma unroll
    for (int poly = 0; poly < 2; poly++) {
        T v[16];
#pragma unroll
        for (int i = 0; i < 16; i++) v[i] = (poly ? a1 : a0)[i];
        row_inv(ar, v, tab, twi, lds, rho, j);
        u64 *o = uo + (size_t)poly * ext * N;
#pragma unroll
        for (int i = 0; i < 16; i++) o[16 * i] = ar.store_ws_inv(v[i]);
    }
}

// grid (8 * ceil(4 TILES * ext / 8) * ceil(n_grp / waves)), 64 waves threads: the rotations of a tile of four rows of one limb run next to each other on one XCD
// (block b runs on XCD b % 8), whose L2 then serves the digits that several rotations of one ciphertext read and the keys
// that several ciphertexts read.
// GROUP: the block adds the inner products of `members` consecutive descriptors (rotations of one ciphertext: same digits,
// their own Galois element and key) before the inverse pass, so that the group is brought back to the ciphertext basis
// by one inverse transform and one ModDown; n_grp then counts groups.
template <int S, bool RAW, bool GROUP, class W>
__global__ __launch_bounds__((RAW ? 64 : 64 * INNER_WAVES), (RAW ? 2 : InnerShape<GROUP, W>::PER_SIMD)) void k_ks16_inner(
    Ks16Const kc, const RotDesc *desc, const PrimeConst *pcs, const u64 *tw_all, u64 *u, int members, u32 n_grp, u32 waves) {
    HIP_DYNAMIC_SHARED(InnerLds, lds)
    constexpr u32 TILES4 = 4 * Ring<S>::TILES;
    constexpr int C = InnerShape<GROUP, W>::VALUES;
    const int ext = kc.l1 + kc.K;
    const u32 wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n_blk = (n_grp + waves - 1) / waves;
    const u32 k = blockIdx.x >> 3, q = k / n_blk * 8 + (blockIdx.x & 7), grp = k % n_blk * waves + wave;
    if (q >= TILES4 * ext || grp >= n_grp) return;
    const int e = ext - 1 - (int)(q / TILES4), prime = ks_ext_prime(e, kc.l1, kc.L);  // the special limbs, which take longer, first
    const PrimeConst pc = load_prime(pcs, prime);
    if (e < kc.l1) inner_body<S, RAW, GROUP, C, ArithFp>(kc, desc, pc, tw_all, u, prime, e, members, grp, q % TILES4, lds[wave].row, lds[wave].tw1);
    else inner_body<S, RAW, GROUP, C, W>(kc, desc, pc, tw_all, u, prime, e, members, grp, q % TILES4, lds[wave].row, lds[wave].tw1);
}

// ------------------------------------------------ the same for few rotations: a wave to each digit
// Where the waves of the form above (RAW) do not fill the chip, their serial chain of beta + 1 row passes and two inverse ones is what
// takes the time.  Here a block takes four rows of one limb of one rotation, each of its waves the row pass and the two products of one digit (the
// last one P * c0); the products meet in LDS, where the automorphism is applied, and two waves run an inverse row pass each.
#define INNER_SPLIT_WAVES 5  // up to four digits
template <int S, class A>
__device__ __forceinline__ void inner_split_body(const Ks16Const &kc, const RotDesc *desc, const PrimeConst &pc, const u64 *tw_all, u64 *u, int prime, int e, u32 grp,
                                                 u32 tile, u32 wave, u64 (*lds)[ROW_LDS], ulonglong2 *tw1) {
    typedef Ring<S> R;
    typedef RowMap<S> M;
    typedef Inner<A> I;
    typedef typename A::T T;
    constexpr size_t N = R::N;
    const int lane = threadIdx.x & 63, rho = lane >> 4, j = lane & 15;
    const int l1 = kc.l1, ext = l1 + kc.K, beta = kc.beta, nd = e < l1 ? beta + 1 : beta;  // P * c0 follows the digits
    const u64 *tw = tw_all + (size_t)prime * 4 * N;
    A ar;
    ar.init(pc);
    const RotDesc d = load_desc(desc, grp);
    const u32 rs = tile * 4 + rho, r = M::row(d.g_inv * M::exponent(rs)), carry = M::carry(r, d.g);
    T *own = (T *)lds[wave];
    T p1[16];
    if ((int)wave < nd) {
        const u64 *src = d.digits + (size_t)((int)wave * ext + e) * N + tile * 1024;
        const u32 row_off = (rho * 256 + j) * 8, reg_off = reg_pos(0, lane) * 8;
        T v[16];
        auto ld = [](const u64 *base, u32 off) { return *(decltype(as_global(base)))((decltype(as_global((const char *)base)))as_global(base) + off); };
        auto ld_pair = [](const u64 *base, u32 off) { return *(__attribute__((address_space(1))) const word_pair *)((decltype(as_global((const char *)base)))as_global(base) + off); };
        row_table_to_lds(tw1, tw, tw + N, R::ROWS + rs, rho, j);
        TwRegs tw2;
        tw2.load(tw, tw + N, N, rs, j);
#pragma unroll
        for (int i = 0; i < 16; i++) v[i] = A::from_bits(ld(src + 16 * i, row_off));
        wave_lds_fence();
        row_fwd<true>(ar, v, tw1 + rho * 16, tw2, lds[wave], rho, j);
        if ((int)wave < beta) {
            const size_t kstride = (size_t)(kc.L + kc.K) * N;
            const u64 *key = d.key + 2 * wave * kstride + (size_t)prime * N + tile * 1024;
#pragma unroll
            for (int h = 0; h < 16; h += 4) {
                word_pair k0[2], k1[2];
#pragma unroll
                for (int i = 0; i < 2; i++) {
                    k0[i] = ld_pair(key + reg_pos(h + 2 * i, 0), reg_off);
                    k1[i] = ld_pair(key + kstride + reg_pos(h + 2 * i, 0), reg_off);
                }
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const u64 x = ar.store_ws_fwd(v[h + i]);
                    T p0 = 0;
                    p1[h + i] = 0;
                    I::mac(ar, p0, x, k0[i / 2][i & 1]);
                    I::mac(ar, p1[h + i], x, k1[i / 2][i & 1]);
                    own[rpad(rho * 256 + 16 * j + h + i)] = p0;
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < 16; i++) {
                T p0 = 0;
                I::add(p0, ar.store_ws_fwd(v[i]));
                own[rpad(rho * 256 + 16 * j + i)] = p0;
            }
        }
    }
    T a[16];
    // value i of lane j, position p = 16 j + i of the output row with brev8(p) = brev4(j) + 16 brev4(i), comes from brev8(g brev8(p) + carry)
    auto sum = [&](int n) {
        const u32 first = d.g * (__brev((u32)j) >> 28) + carry;
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const u32 brev4_i = (i & 1) * 8 + (i & 2) * 2 + (i & 4) / 2 + (i & 8) / 8;
            const int at = rpad(rho * 256 + brev8(first + d.g * (16 * brev4_i)));
            a[i] = ((const T *)lds[0])[at];
            for (int w = 1; w < n; w++) a[i] = I::plus_lazy(ar, a[i], ((const T *)lds[w])[at]);
            I::fold(ar, a[i]);
        }
    };
    __syncthreads();
    if (wave == 0) sum(nd);
    __syncthreads();
    if ((int)wave < beta) {
#pragma unroll
        for (int i = 0; i < 16; i++) own[rpad(rho * 256 + 16 * j + i)] = p1[i];
    }
    __syncthreads();
    if (wave == 1) sum(beta);
    __syncthreads();
    if (wave < 2) {
        tw += 2 * N;
        row_table_to_lds(tw1, tw, tw + N, R::ROWS + r, rho, j);
        TwRegs twi;
        twi.load(tw, tw + N, N, r, j);
        wave_lds_fence();
        row_inv(ar, a, tw1 + rho * 16, twi, lds[wave], rho, j);
        u64 *o = u + ((size_t)(grp * 2 + wave) * ext + e) * N + (size_t)r * 256 + j;
#pragma unroll
        for (int i = 0; i < 16; i++) o[16 * i] = ar.store_ws_inv(a[i]);
    }
}
// grid (8 * ceil(4 TILES * ext / 8) * n_rot), 64 (beta + 1) threads (at least two waves)
template <int S, class W>
__global__ __launch_bounds__((64 * INNER_SPLIT_WAVES), (std::is_same<W, ArithInt>::value ? 3 : 4)) void k_ks16_inner_split(Ks16Const kc, const RotDesc *desc, const PrimeConst *pcs, const u64 *tw_all, u64 *u,
                                                                                u32 n_rot) {
    __shared__ u64 lds[INNER_SPLIT_WAVES][ROW_LDS];
    __shared__ ulonglong2 tw1[INNER_SPLIT_WAVES][4 * 16];
    constexpr u32 TILES4 = 4 * Ring<S>::TILES;
    const int ext = kc.l1 + kc.K;
    const u32 wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const u32 k = blockIdx.x >> 3, q = k / n_rot * 8 + (blockIdx.x & 7), grp = k % n_rot;
    if (q >= TILES4 * ext) return;
    const int e = ext - 1 - (int)(q / TILES4), prime = ks_ext_prime(e, kc.l1, kc.L);
    const PrimeConst pc = load_prime(pcs, prime);
    if (e < kc.l1) inner_split_body<S, ArithFp>(kc, desc, pc, tw_all, u, prime, e, grp, q % TILES4, wave, lds, tw1[wave]);
    else inner_split_body<S, W>(kc, desc, pc, tw_all, u, prime, e, grp, q % TILES4, wave, lds, tw1[wave]);
}

// ------------------------------------------------------ inverse column pass + ModDown
// Special limb k of one column tile: inverse column pass and the centred residue of u (P/p_k)^-1, as hi * 2^30 + lo (lo in
// [0, 2^30), hi signed).
__device__ __forceinline__ int64_t special_centred(const ArithWide &ar, int64_t v, const Ks16Const &kc, int k) {
    return ar.centred(ar.mul(v, as_const(kc.down_p)[2 * k], as_const(kc.down_p)[2 * k + 1]));
}
__device__ __forceinline__ int64_t special_centred(const ArithFp &ar, double v, const Ks16Const &kc, int k) {
    return (int64_t)ar.mid(ar.mulmod(v, as_const(kc.down_p_fp)[2 * k], as_const(kc.down_p_fp)[2 * k + 1]));
}
__device__ __forceinline__ int64_t special_centred(const ArithInt &ar, u64 v, const Ks16Const &kc, int k) {
    const u64 y = mul_shoup(v, as_const(kc.down_p)[2 * k], as_const(kc.down_p)[2 * k + 1], ar.q);
    return y > ar.q / 2 ? (int64_t)y - (int64_t)ar.q : (int64_t)y;
}
// y_k as two int32 words
__device__ __forceinline__ u64 special_word(int64_t z) { return ((u64)(u32)(int32_t)(z >> 30) << 32) | (u32)(z & 0x3fffffff); }
// The special limbs of few rotations, a block each: y_k in place of the limb of the accumulator, at the rows where the ciphertext limbs of a
// column tile have theirs.  grid (TILES, 2 * K, n_rot / members)
template <int S, class W>
__global__ __launch_bounds__(KS_THREADS, 4) void k_ks16_specials(Ks16Const kc, const PrimeConst *pcs, const u64 *tw_all, u64 *u) {
    typedef Ring<S> R;
    constexpr size_t N = R::N;
    __shared__ ColLdsOne sh;
    const int tid = threadIdx.x, c = R::col(tid), jj = R::grp(tid), poly = blockIdx.y / kc.K, k = blockIdx.y - poly * kc.K, ext = kc.l1 + kc.K;
    u64 *at = u + (((size_t)blockIdx.z * 2 + poly) * ext + kc.l1 + k) * N + (size_t)blockIdx.x * R::COLS;
    const u64 *tw = tw_all + (size_t)(kc.L + k) * 4 * N + 2 * N;
    u32 tidx = 0;
    const int tplace = col_tab_index<S>(tid, &tidx);
    if (tplace >= 0) sh.tab[tplace] = make_ulonglong2(tw[tidx], tw[N + tidx]);
    W ar;
    ar.init(load_prime(pcs, kc.L + k));
    typename W::T v[16];
#pragma unroll
    for (int i = 0; i < 16; i++) v[i] = W::from_bits(ld_off(at + i * 256, (16 * jj * 256 + c) * 8));
    __syncthreads();
    cols_inv_tab<S>(ar, v, sh.tab, sh.tile, c, jj);  // (its barrier comes after every thread's reads of the tile)
#pragma unroll
    for (int i = 0; i < 16; i++) st_off(at + R::row(0, i) * 256, (R::row(jj, 0) * 256 + c) * 8, special_word(special_centred(ar, v[i], kc, k)));
}
// grid (TILES, 2 * parts, n_rot / members): a block brings the special limbs of one column tile of one accumulator back
// and then `per` ciphertext limbs.  K: the number of special primes.  READY: k_ks16_specials has brought them back (W has no say then).
template <int S, class W, int K, bool READY>
__global__ __launch_bounds__(KS_THREADS, 2) void k_ks16_icols(Ks16Const kc, const RotDesc *desc, const PrimeConst *pcs, const u64 *tw_all, const u64 *u,
                                                              int limb_stride_out, int members, int per) {
    typedef Ring<S> R;
    constexpr size_t N = R::N;
    __shared__ ColLds sh;
    const int tid = threadIdx.x, c = R::col(tid), jj = R::grp(tid);
    const int l1 = kc.l1, ext = l1 + K;
    const int parts = (l1 + per - 1) / per, poly = blockIdx.y / parts, i0 = (blockIdx.y - poly * parts) * per, i1 = min(l1, i0 + per);
    const u64 *src = u + ((size_t)blockIdx.z * 2 + poly) * ext * N + (size_t)blockIdx.x * R::COLS;
    const u32 off_in = (16 * jj * 256 + c) * 8, off_out = (R::row(jj, 0) * 256 + c) * 8;
    u32 tidx = 0;
    const int tplace = col_tab_index<S>(tid, &tidx);
    ulonglong2 tnext;
    u64 nv[16];
    // step t of the walk: special limb t for t < K, then ciphertext limb i0 + t - K
    const int n_steps = K + i1 - i0;
    auto fetch = [&](int t) {
        const int limb = t < K ? l1 + t : i0 + t - K;
        const u64 *tw = tw_all + (size_t)ks_ext_prime(limb, l1, kc.L) * 4 * N + 2 * N;
        tnext = make_ulonglong2(tw[tidx], tw[N + tidx]);
#pragma unroll
        for (int i = 0; i < 16; i++) nv[i] = ld_off(src + (size_t)limb * N + i * 256, off_in);
    };
    auto put_tab = [&](int buf) {
        if (tplace >= 0) sh.tab[buf][tplace] = tnext;
    };
    fetch(READY ? K : 0);
    put_tab(READY ? K % 3 : 0);
    u64 y[K][16];
    if (READY) {
#pragma unroll
        for (int k = 0; k < K; k++)
#pragma unroll
            for (int i = 0; i < 16; i++) y[k][i] = ld_off(src + (size_t)(l1 + k) * N + R::row(0, i) * 256, off_out);
    }
    __syncthreads();
    auto special = [&](u64 *yk, int k) {
        W ar;
        ar.init(load_prime(pcs, kc.L + k));
        typename W::T v[16];
#pragma unroll
        for (int i = 0; i < 16; i++) v[i] = W::from_bits(nv[i]);
        fetch(k + 1);
        put_tab((k + 1) % 3);
        cols_inv_tab<S>(ar, v, sh.tab[k % 3], sh.tile[k & 1], c, jj);
#pragma unroll
        for (int i = 0; i < 16; i++) {
            yk[i] = special_word(special_centred(ar, v[i], kc, k));
            keep_narrow(yk[i]);
        }
    };
    if constexpr (!READY) {
        special(y[0], 0);
        if constexpr (K > 1) special(y[1], 1);
        if constexpr (K > 2) special(y[2], 2);
        if constexpr (K > 3) special(y[3], 3);
    }
    const RotDesc dl = load_desc(desc, blockIdx.z * members);  // the group's first descriptor carries the destination
    auto out_at = [&](u64 *out, int i) { return (decltype(as_global(out)))((decltype(as_global((char *)out)))as_global(out + R::row(0, i) * 256) + off_out); };
    int tcur = K % 3;
#pragma unroll 1
    for (int t = K; t < n_steps; t++) {
        const int limb = i0 + t - K;
#pragma unroll
        for (int k = 0; k < K; k++)
#pragma unroll
            for (int i = 0; i < 16; i++) keep_narrow(y[k][i]);
        const PrimeConst pc = load_prime(pcs, limb);
        ArithFp ar;
        ar.init(pc);
        double v[16];
#pragma unroll
        for (int i = 0; i < 16; i++) v[i] = as_f64(nv[i]);
        if (t + 1 < n_steps) fetch(t + 1);
        const int tnxt = tcur == 2 ? 0 : tcur + 1;
        put_tab(tnxt);
        cols_inv_tab<S>(ar, v, sh.tab[tcur], sh.tile[t & 1], c, jj);
        tcur = tnxt;
        const double sc = as_const(kc.down_q)[2 * limb], sc_p = as_const(kc.down_q)[2 * limb + 1];
        u64 *out = dl.out + ((size_t)poly * limb_stride_out + limb) * N + (size_t)blockIdx.x * R::COLS;
        // sum_k lo_k p_k^-1 + hi_k 2^30 p_k^-1 over split constants: four multiply-adds per special limb, one reduction
        // (two modular products per special limb in fp64 took 2.5 times the instructions); |sums| < 2^59
#pragma unroll
        for (int h = 0; h < 16; h += 4) {
            int64_t a0[4], a1[4];
#pragma unroll
            for (int k = 0; k < K; k++) {
                const u64 hl = as_const(kc.down_h)[(limb * K + k) * 2], hh = as_const(kc.down_h)[(limb * K + k) * 2 + 1];
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const int lo = (int)(u32)y[k][h + i], hi = (int)(y[k][h + i] >> 32);
                    a0[i] = mad_i(hi, (int)(u32)hh, k ? mad_i(lo, (int)(u32)hl, a0[i]) : mul_i(lo, (int)(u32)hl));
                    a1[i] = mad_i(hi, (int)(hh >> 32), k ? mad_i(lo, (int)(hl >> 32), a1[i]) : mul_i(lo, (int)(hl >> 32)));
                }
            }
            u64 w[4];
#pragma unroll
            for (int i = 0; i < 4; i++) w[i] = ar.canon(ar.mulmod(v[h + i], sc, sc_p) - ar.reduce25_long(a1[i], a0[i]));
            if (dl.accumulate) {
                // out <- out + result.  `out` may be the rotation's own source (every read of the source happened in the
                // raise kernels, which have finished), which turns t <- t + Rot(t; r) into one pass
#pragma unroll
                for (int i = 0; i < 4; i++) w[i] = add_mod(*out_at(out, h + i), w[i], pc.q);
            }
#pragma unroll
            for (int i = 0; i < 4; i++) *out_at(out, h + i) = w[i];
        }
    }
}

// ---------------------------------------------------------------- launchers of one ring
// Limbs per block of the two column kernels: all of them where that still gives every CU four blocks (y is then formed
// once), otherwise as few as it takes to get there.  blocks: blocks at one limb-walk each; limbs: length of the walk.
static int limbs_per_block(long blocks, int limbs) {
    const long want = 1024;
    if (blocks >= want) return limbs;
    const long parts = (want + blocks - 1) / blocks;
    return (int)((limbs + parts - 1) / parts);
}

// Few rotations, which do not fill the chip.  Whole calls of ensi_rotate, without and with each form, in us, on 2^16 with 10 + 3 limbs (and 16 + 4),
// 2^14 with 6 + 2 and 2^12 with 3 + 1:
// Raise with a limb to a block (k_ks16_fcols_one), where the blocks of a limb each are more than the two to a CU that the walking form
// has room for, and up to three times as many: one rotation 91, 82 (118, 116); two 127, 128; 2^14: no difference.
#define FCOLS_ONE_MIN 512
#define FCOLS_ONE_MAX 1536
// Special limbs first (k_ks16_specials), where otherwise several blocks would bring the same ones back, by column tiles of accumulators: one
// rotation 91, 84 (118, 105), two 127, 113 (210, 175), eight 348, 343, 16 578, 585; 2^14: one 45, 45, 24 141, 133; a single special prime
// is not worth the launch (2^12: 36, 39).
#define SPECIALS_FIRST_MAX 256
// Inner products with a wave to each digit (k_ks16_inner_split), by waves of the form with one to a tile: on 2^12 one rotation 36, 30, 32
// 55, 43, 64 (1024 waves) 65, 67; on 2^14 four 55, 53, eight 75, 79; on 2^16 one with 5 limbs (512) 57, 57, with 10 (832) 91, 102.
#define INNER_SPLIT_MAX 512

// Calls f with the arithmetic of the special primes.
template <class F>
static void special_dispatch(const ensi_ctx *ctx, F f) {
    if (ctx->special_kind == PRIME_WIDE) f(ArithWide{});
    else if (ctx->special_kind == PRIME_FP) f(ArithFp{});
    else f(ArithInt{});
}

template <int S>
void ks16_raise(ensi_ctx *ctx, const Ks16Const &kc, const u64 *ct_base, size_t ct_stride_words, int limb_stride, int n_ct, u64 *dig, bool rows,
                       hipStream_t st) {
    const int ext = kc.l1 + kc.K, n_rows = kc.beta * ext + kc.l1;
    special_dispatch(ctx, [&](auto w) {
        constexpr int TILES = Ring<S>::TILES;
        typedef decltype(w) W;
        {
            ScopedTimer t(ctx, "ks_modup_fcols", st);
            const long limbs = (long)TILES * n_rows * n_ct;
            if (limbs > FCOLS_ONE_MIN && limbs <= FCOLS_ONE_MAX) {
                hipLaunchKernelGGL((k_ks16_fcols_one<S, W>), dim3(TILES, n_rows, n_ct), dim3(KS_THREADS), 0, st, kc, ctx->d_pc, ctx->d_tw, ct_base, ct_stride_words,
                                   limb_stride, dig);
            } else {
                const int per = limbs_per_block((long)TILES * (kc.beta + 1) * n_ct, ext);
                hipLaunchKernelGGL((k_ks16_fcols<S, W>), dim3(TILES, kc.beta * ((ext + per - 1) / per) + (kc.l1 + per - 1) / per, n_ct), dim3(KS_THREADS), 0, st, kc,
                                   ctx->d_pc, ctx->d_tw, ct_base, ct_stride_words, limb_stride, dig, per);
            }
        }
        if (rows) {
            ScopedTimer t(ctx, "ks_frows", st);
            hipLaunchKernelGGL((k_ks16_frows<S, W>), dim3(4 * TILES * n_rows * ((n_ct + KS_FROWS_GROUP - 1) / KS_FROWS_GROUP)), dim3(64), 0, st, kc, ctx->d_pc,
                               ctx->d_tw, dig, n_ct);
        }
    });
}

template <int S>
void ks16_switch(ensi_ctx *ctx, const Ks16Const &kc, const RotDesc *d_desc, int n_rot, u64 *u, int limb_stride_out, bool raw, hipStream_t st,
                        int members) {
    // n_rot descriptors in groups of `members` (1: every rotation on its own); u is indexed by group
    const int n_grp = n_rot / members, ext = kc.l1 + kc.K;
    special_dispatch(ctx, [&](auto w) {
        constexpr int TILES = Ring<S>::TILES;
        typedef decltype(w) W;
        {
            ScopedTimer t(ctx, "ks_inner", st);
            auto inner = [&](auto raw_, auto group_) {
                const unsigned waves = decltype(raw_)::value || n_grp < INNER_WAVES_MIN ? 1 : INNER_WAVES;
                const unsigned blocks = (4u * TILES * ext + 7) / 8 * 8 * ((n_grp + waves - 1) / waves);
                hipLaunchKernelGGL((k_ks16_inner<S, decltype(raw_)::value, decltype(group_)::value, W>), dim3(blocks), dim3(64 * waves), waves * sizeof(InnerLds), st, kc,
                                   d_desc, ctx->d_pc, ctx->d_tw, u, members, (u32)n_grp, waves);
            };
            if (raw && kc.beta < INNER_SPLIT_WAVES && 4l * TILES * ext * n_rot <= INNER_SPLIT_MAX)
                hipLaunchKernelGGL((k_ks16_inner_split<S, W>), dim3((4u * TILES * ext + 7) / 8 * 8 * n_rot), dim3(64 * (kc.beta + 1)), 0, st, kc, d_desc, ctx->d_pc,
                                   ctx->d_tw, u, (u32)n_rot);
            else if (raw) inner(std::true_type(), std::false_type());
            else if (members > 1) inner(std::false_type(), std::true_type());
            else inner(std::false_type(), std::false_type());
        }
        ScopedTimer t(ctx, "ks_icols_moddown", st);
        const int per = limbs_per_block((long)TILES * 2 * n_grp, kc.l1);
        const bool ready = kc.K > 1 && per < kc.l1 && (long)TILES * 2 * n_grp <= SPECIALS_FIRST_MAX;
        if (ready) hipLaunchKernelGGL((k_ks16_specials<S, W>), dim3(TILES, 2 * kc.K, n_grp), dim3(KS_THREADS), 0, st, kc, ctx->d_pc, ctx->d_tw, u);
        auto icols = [&](auto k) {
            if (ready)
                hipLaunchKernelGGL((k_ks16_icols<S, ArithFp, decltype(k)::value, true>), dim3(TILES, 2 * ((kc.l1 + per - 1) / per), n_grp), dim3(KS_THREADS), 0, st, kc,
                                   d_desc, ctx->d_pc, ctx->d_tw, u, limb_stride_out, members, per);
            else
                hipLaunchKernelGGL((k_ks16_icols<S, W, decltype(k)::value, false>), dim3(TILES, 2 * ((kc.l1 + per - 1) / per), n_grp), dim3(KS_THREADS), 0, st, kc, d_desc,
                                   ctx->d_pc, ctx->d_tw, u, limb_stride_out, members, per);
        };
        if (kc.K == 1) icols(std::integral_constant<int, 1>{});
        else if (kc.K == 2) icols(std::integral_constant<int, 2>{});
        else if (kc.K == 3) icols(std::integral_constant<int, 3>{});
        else icols(std::integral_constant<int, 4>{});
    });
}
