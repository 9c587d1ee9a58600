// The client's side on the rings N = 2^12 .. 2^16 with ciphertext primes below 2^50: encode, encrypt, decrypt and decode on
// the passes of the register transform (ntt16_core.h), so that a batch is a handful of launches.
//
// Encoding (paper, Preliminaries: SIMD Encoding).  Slot j is the value of m(X) at exp(i pi 5^j / N), and both directions are
// the length-2N transform of kernels.hip -- with the same butterflies on the same numbers in the same order, so that
// coefficients and slots are those of that transform to the last bit, on every ring and at every scale.  What is left
// out are butterflies on zeros and on outputs that nobody reads.  The exponents 5^j mod 2N, j < n = N/2, are exactly those
// congruent to 1 modulo 4; with 5^j = 4k + 1 and the pass of stride s pairing the elements p and p + N/s:
//   encode  Every pass keeps an element's p modulo 4, so that only the n elements with p = 4 p' + 1 ever differ from zero until
//           the last two passes, which take x = (re, im) of those to the coefficients t and t + n.
//   decode  The first pass has one input per butterfly, the second is read at its even outputs alone; the others are n points.
// The n points are cut as t = 256 r + c, k = k1 + R2 k2 (R2 = N / 512 rows): the passes over 256 elements of a row and those
// over the R2 rows of a column, each on 2048 values in LDS.
//
// These kernels are small against the copies from and to host memory beside them; what counts is their number.
#include "common.h"
#include "ntt16_core.h"

#define CL_THREADS 256

// ------------------------------------------------------------------ complex transforms in LDS
// sine of exponent e of the table of cosines, as the transform's passes read it
template <int N>
__device__ __forceinline__ double sine(const double *cos_tab, u32 e) { return cos_tab[(e - N / 2) & (2 * N - 1)]; }
// Consecutive passes of the transform on 2048 / LEN sequences of LEN points at once (element t of sequence b at x[t * B + b],
// B = 2048 / LEN).  The butterfly of element p in the pass of local stride s has the exponent base(b) s + STEP p s; a pass's
// exponentials, scattered over the table, are requested before the barrier that precedes it.
// Returns the buffer that holds the result; every thread may read it.
template <int N, int LEN, int STEP, class F>
__device__ __forceinline__ double2 *lds_passes(double2 *x, double2 *y, const double *cos_tab, int tid, F base) {
    constexpr int B = 2048 / LEN;
    double2 tw[4];
    auto fetch = [&](int s) {
#pragma unroll
        for (int m = 0; m < 4; m++) {
            const int w = tid + CL_THREADS * m, t = w / B;
            const u32 e = (u32)base(w % B) * s + (u32)(t - (t & (s - 1))) * STEP;
            tw[m] = make_double2(cos_tab[e], sine<N>(cos_tab, e));
        }
    };
    fetch(1);
    __syncthreads();
#pragma unroll 1
    for (int s = 1; s < LEN; s *= 2) {
#pragma unroll
        for (int m = 0; m < 4; m++) {
            const int w = tid + CL_THREADS * m, b = w % B, t = w / B;
            const int q = t & (s - 1), idx = t - q;
            fft_butterfly(x[t * B + b], x[(t + LEN / 2) * B + b], tw[m].x, tw[m].y, y[(q + 2 * idx) * B + b], y[(q + 2 * idx + s) * B + b]);
        }
        if (2 * s < LEN) fetch(2 * s);
        __syncthreads();
        double2 *h = x;
        x = y;
        y = h;
    }
    return x;
}

// ------------------------------------------------------------------ encode
// grid (R2 / 8, n_pt): eight rows k1.  ws: [n_pt][R2][256]
template <int S>
__global__ __launch_bounds__(CL_THREADS) void k_cl_enc_rows(const double *slots, int n_slots, int slot0, int slot_step, int y0, const u32 *slot_of_k,
                                                            const double *cos_tab, double2 *ws) {
    constexpr int N = Ring<S>::N, R2 = N / 512;
    __shared__ double2 buf[2][2048];
    const int tid = threadIdx.x, y = y0 + blockIdx.y, first = slot0 + y * slot_step, k1 = blockIdx.x * 8;
    const double *z = slots + (size_t)blockIdx.y * n_slots;
#pragma unroll
    for (int m = 0; m < 8; m++) {
        const int w = tid + CL_THREADS * m, row = w & 7, k2 = w >> 3;
        const int j = (int)slot_of_k[k1 + row + R2 * k2] - first;
        buf[0][w] = make_double2(j >= 0 && j < n_slots ? z[j] : 0.0, 0.0);
    }
    const double2 *f = lds_passes<N, 256, 4 * R2>(buf[0], buf[1], cos_tab, tid, [&](int row) { return 4 * (k1 + row) + 1; });
#pragma unroll
    for (int row = 0; row < 8; row++) ws[((size_t)blockIdx.y * R2 + k1 + row) * 256 + tid] = f[tid * 8 + row];
}
// grid (TILES, n_pt): one tile of columns.  out: [n_pt][limbs][N] canonical residues
template <int S>
__global__ __launch_bounds__(CL_THREADS) void k_cl_enc_cols(const double2 *ws, double factor, int limbs, const PrimeConst *pcs, const double *cos_tab,
                                                            u64 *out) {
    typedef Ring<S> R;
    constexpr int N = R::N, R2 = N / 512;
    __shared__ double2 buf[2][2048];
    const int tid = threadIdx.x;
#pragma unroll
    for (int m = 0; m < 8; m++) {
        const int w = tid + CL_THREADS * m, c = w % R::COLS, k1 = w / R::COLS;
        buf[0][w] = ws[((size_t)blockIdx.y * R2 + k1) * 256 + blockIdx.x * R::COLS + c];
    }
    const double2 *f = lds_passes<N, R2, 1024>(buf[0], buf[1], cos_tab, tid, [](int) { return 256; });
    int64_t v[16];
#pragma unroll
    for (int m = 0; m < 8; m++) {
        // the last two passes: one input of each butterfly is zero
        double2 even, odd;
        fft_butterfly(f[tid + CL_THREADS * m], make_double2(0.0, 0.0), cos_tab[N / 2], cos_tab[0], even, odd);
        v[2 * m] = round_coeff(even.x * factor);
        v[2 * m + 1] = round_coeff(odd.x * factor);
    }
    for (int l = 0; l < limbs; l++) {
        ArithFp ar;
        ar.init(load_prime(pcs, l));
        auto residue = [&](int64_t x) { return ar.canon(ar.mid((double)(int)(x >> 32) * 4294967296.0) + (double)(u32)x); };
        u64 *o = out + ((size_t)blockIdx.y * limbs + l) * N;
#pragma unroll
        for (int m = 0; m < 8; m++) {
            const int w = tid + CL_THREADS * m, t = w / R::COLS * 256 + blockIdx.x * R::COLS + w % R::COLS;
            o[t] = residue(v[2 * m]);
            o[t + N / 2] = residue(v[2 * m + 1]);
        }
    }
}

// ------------------------------------------------------------------ encrypt
// Forward column pass of n polynomials of small integers at every limb.  grid (TILES, limbs, n); ws: [n][limbs][N] doubles
template <int S>
__global__ __launch_bounds__(CL_THREADS) void k_cl_fcols_small(const int8_t *small, const PrimeConst *pcs, const u64 *tw_all, u64 *ws) {
    typedef Ring<S> R;
    constexpr size_t N = R::N;
    __shared__ u64 lds[4096];
    const int c = R::col(threadIdx.x), jj = R::grp(threadIdx.x), limb = blockIdx.y;
    ArithFp ar;
    ar.init(load_prime(pcs, limb));
    const u64 *tw = tw_all + (size_t)limb * 4 * N;
    const int8_t *in = small + (size_t)blockIdx.z * N + blockIdx.x * R::COLS + c;
    double v[16];
#pragma unroll
    for (int i = 0; i < 16; i++) v[i] = (double)in[R::row(jj, i) * 256];
    cols_fwd_regs<S>(ar, v, tw, tw + N, lds, c, jj);
    u64 *o = ws + ((size_t)blockIdx.z * gridDim.y + limb) * N + (size_t)blockIdx.x * R::COLS + c;
#pragma unroll
    for (int i = 0; i < 16; i++) o[(size_t)(16 * jj + i) * 256] = ar.store_ws_cols(v[i]);
}
// Forward row pass, product with POLYS key polynomials (key: limb `limb` of polynomial p at (p * key_limbs + limb) * N, in
// position order, Montgomery residues: the factor 2^-64 they owe is part of the constant that the column pass behind this
// kernel scales by) and inverse row pass of each product.  A wave runs four rows of one limb of one of the n polynomials.  The
// twiddles of both directions and the key words are five times the bytes of the rows themselves: the waves of the n polynomials
// that share them run next to each other on one XCD (block b runs on XCD b % 8) and find them in its L2.  (Polynomials launched
// one after the other fetched 540 MB for 10 x 16 limbs: 116 us, then 94.  Waves that keep the twiddles for five polynomials in registers: 100.)
// grid (8 * ceil(4 TILES * limbs / 8) * n); in: [n][limbs][N], out: [n][POLYS][limbs][N] doubles (may be the same array if
// POLYS is 1)
template <int S, int POLYS>
__global__ __launch_bounds__(64, 2) void k_cl_rows_key(const u64 *in, const u64 *key, int key_limbs, int limbs, u32 n, const PrimeConst *pcs,
                                                       const u64 *tw_all, u64 *out) {
    typedef Ring<S> R;
    constexpr size_t N = R::N;
    constexpr u32 TILES4 = 4 * R::TILES;
    __shared__ u64 lds[ROW_LDS];
    __shared__ ulonglong2 tw1[2][4 * 16];
    const u32 k = blockIdx.x >> 3, q = k / n * 8 + (blockIdx.x & 7), z = k % n;
    if (q >= TILES4 * limbs) return;
    const int lane = threadIdx.x, rho = lane >> 4, j = lane & 15, limb = q / TILES4;
    const u32 r = q % TILES4 * 4 + rho;
    ArithFp ar;
    ar.init(load_prime(pcs, limb));
    const u64 *twf = tw_all + (size_t)limb * 4 * N, *twi = twf + 2 * N;
    double v[16];
    const u64 *src = in + ((size_t)z * limbs + limb) * N + (size_t)r * 256 + j;
#pragma unroll
    for (int i = 0; i < 16; i++) v[i] = __longlong_as_double((long long)src[16 * i]);
    row_table_to_lds(tw1[0], twf, twf + N, R::ROWS + r, rho, j);
    row_table_to_lds(tw1[1], twi, twi + N, R::ROWS + r, rho, j);
    TwRegs tw2;
    tw2.load(twf, twf + N, N, r, j);
    // The key's rows are read like the polynomial's, a line to sixteen lanes, and brought to the places of the products through LDS: read
    // in place every load touches 64 lines (10 x 16 limbs, two polynomials: 91 to 95 us so, now 86; one polynomial of few limbs waits for
    // the exchange instead, 12 us so and 14).
    u64 kw[16];
    auto fetch_key = [&](int p) {
        const u64 *kp = key + ((size_t)p * key_limbs + limb) * N + (size_t)r * 256 + j;
#pragma unroll
        for (int i = 0; i < 16; i++) kw[i] = kp[16 * i];
    };
    if (POLYS > 1) fetch_key(0);
    wave_lds_fence();
    row_fwd<true>(ar, v, tw1[0] + rho * 16, tw2, lds, rho, j);
#pragma unroll
    for (int i = 0; i < 16; i++) v[i] = ar.mid(v[i]);
    tw2.load(twi, twi + N, N, r, j);
#pragma unroll
    for (int p = 0; p < POLYS; p++) {
        if (POLYS > 1) {
#pragma unroll
            for (int i = 0; i < 16; i++) lds[rpad(rho * 256 + j + 16 * i)] = kw[i];
            wave_lds_fence();
#pragma unroll
            for (int i = 0; i < 16; i++) kw[i] = lds[rpad(rho * 256 + 16 * j + i)];
            wave_lds_fence();
        } else {
            const u64 *kp = key + ((size_t)p * key_limbs + limb) * N + (size_t)r * 256 + 16 * j;
#pragma unroll
            for (int i = 0; i < 16; i++) kw[i] = kp[i];
        }
        double x[16];
#pragma unroll
        for (int i = 0; i < 16; i++) x[i] = ar.mid(ar.mulmod_np(v[i], ar.load(kw[i])));
        if (p + 1 < POLYS) fetch_key(p + 1);
        row_inv(ar, x, tw1[1] + rho * 16, tw2, lds, rho, j);
        u64 *o = out + (((size_t)z * POLYS + p) * limbs + limb) * N + (size_t)r * 256 + j;
#pragma unroll
        for (int i = 0; i < 16; i++) o[16 * i] = ar.store_ws_inv(x[i]);
    }
}
// x / (N 2^64) mod p of a value of the row pass above
struct ScaleDown {
    double w, wp;
    __device__ __forceinline__ void init(const ArithFp &ar, const PrimeConst &pc) {
        const acc128 m = {pc.n_inv, 0};
        w = (double)mont_reduce(m, pc.q, pc.qneg_inv);
        wp = w * ar.pinv;
    }
    __device__ __forceinline__ double operator()(const ArithFp &ar, double x) const { return ar.mulmod(ar.mid(x), w, wp); }
};
// Inverse column pass in place, plus the error polynomial and, on the first polynomial, the message: the ciphertext.
// grid (TILES, 2 * limbs, n); errors: e0 of all ciphertexts, then (err_stride further) e1
// As many blocks on a CU as its registers allow: asked for the four that its LDS holds, the rings 2^13 and 2^15 spilled 44 and 40
// (64 x 6 limbs of 2^13 38.4 us, 26 so; 10 x 12 of 2^15 44.5, 31; 10 x 16 of 2^16 89.4, 87).
template <int S>
__global__ __launch_bounds__(CL_THREADS) void k_cl_icols_add(u64 *ct, const int8_t *errors, size_t err_stride, const u64 *pt, int limbs,
                                                             const PrimeConst *pcs, const u64 *tw_all) {
    typedef Ring<S> R;
    constexpr size_t N = R::N;
    __shared__ u64 lds[4096];
    __shared__ __attribute__((aligned(16))) int8_t err[4096];
    const int c = R::col(threadIdx.x), jj = R::grp(threadIdx.x), poly = blockIdx.y / limbs, limb = blockIdx.y - poly * limbs;
    const size_t col = (size_t)blockIdx.x * R::COLS + c;
    const PrimeConst pc = load_prime(pcs, limb);
    ArithFp ar;
    ar.init(pc);
    ScaleDown down;
    down.init(ar, pc);
    const u64 *tw = tw_all + (size_t)limb * 4 * N + 2 * N;
    u64 *g = ct + ((size_t)blockIdx.z * 2 * limbs + blockIdx.y) * N + col;
    const u64 *m = pt + ((size_t)blockIdx.z * limbs + limb) * N + col;
    // The tile's errors, sixteen bytes a thread, pass through LDS: fetched byte by byte where they are added they were waited for
    // one after the other (a wave lived 22 us; 10 x 16 limbs 144 us, now 87).
    double v[16];
    u64 a[16] = {};
#pragma unroll
    for (int i = 0; i < 16; i++) v[i] = __longlong_as_double((long long)g[(size_t)(16 * jj + i) * 256]);
    const int at = threadIdx.x * 16;  // of the tile's 4096 bytes
    const uint4 mine = *(const uint4 *)(errors + poly * err_stride + blockIdx.z * N + (at >> R::LOGC) * 256 + blockIdx.x * R::COLS + (at & (R::COLS - 1)));
    if (poly == 0) {
#pragma unroll
        for (int i = 0; i < 16; i++) a[i] = m[(size_t)R::row(jj, i) * 256];
    }
    *(uint4 *)(err + at) = mine;
    if (S == 0) __syncthreads();  // (on larger rings the pass has a barrier)
    cols_inv_regs<S>(ar, v, tw, tw + N, lds, c, jj);
#pragma unroll
    for (int i = 0; i < 16; i++)
        g[(size_t)R::row(jj, i) * 256] = ar.canon(down(ar, v[i]) + ((double)err[R::row(jj, i) * R::COLS + c] + ar.load(a[i])));
}

// ------------------------------------------------------------------ decrypt
// Forward column pass of c1.  grid (TILES, use, n); ws: [n][use][N]
template <int S>
__global__ __launch_bounds__(CL_THREADS) void k_cl_fcols_c1(const u64 *ct, int limbs_alloc, const PrimeConst *pcs, const u64 *tw_all, u64 *ws) {
    typedef Ring<S> R;
    constexpr size_t N = R::N;
    __shared__ u64 lds[4096];
    const int c = R::col(threadIdx.x), jj = R::grp(threadIdx.x), limb = blockIdx.y;
    const size_t col = (size_t)blockIdx.x * R::COLS + c;
    ArithFp ar;
    ar.init(load_prime(pcs, limb));
    const u64 *tw = tw_all + (size_t)limb * 4 * N, *in = ct + (((size_t)blockIdx.z * 2 + 1) * limbs_alloc + limb) * N + col;
    double v[16];
#pragma unroll
    for (int i = 0; i < 16; i++) v[i] = ar.load(in[(size_t)R::row(jj, i) * 256]);
    cols_fwd_regs<S>(ar, v, tw, tw + N, lds, c, jj);
    u64 *o = ws + ((size_t)blockIdx.z * gridDim.y + limb) * N + col;
#pragma unroll
    for (int i = 0; i < 16; i++) o[(size_t)(16 * jj + i) * 256] = ar.store_ws_cols(v[i]);
}
// Inverse column pass of c1 s on both limbs, + c0, the centred coefficient, and the column part of the decoding transform.
// grid (TILES, n); f: [n][R2][256]
template <int S>
__global__ __launch_bounds__(CL_THREADS) void k_cl_dec_cols(const u64 *ws, int use, const u64 *ct, int limbs_alloc, CrtPair crt, const PrimeConst *pcs,
                                                            const u64 *tw_all, const double *cos_tab, double2 *f) {
    typedef Ring<S> R;
    constexpr int NI = R::N, R2 = NI / 512;
    constexpr size_t N = R::N;
    __shared__ double2 buf[2][2048];  // the column passes use it as a tile of words
    const int tid = threadIdx.x, c = R::col(tid), jj = R::grp(tid);
    const size_t col = (size_t)blockIdx.x * R::COLS + c;
    u64 r[2][16];
#pragma unroll
    for (int limb = 0; limb < 2; limb++) {
        if (limb < use) {
            const PrimeConst pc = load_prime(pcs, limb);
            ArithFp ar;
            ar.init(pc);
            ScaleDown down;
            down.init(ar, pc);
            const u64 *tw = tw_all + (size_t)limb * 4 * N + 2 * N;
            const u64 *in = ws + ((size_t)blockIdx.y * use + limb) * N + col, *c0 = ct + ((size_t)blockIdx.y * 2 * limbs_alloc + limb) * N + col;
            double v[16];
#pragma unroll
            for (int i = 0; i < 16; i++) v[i] = __longlong_as_double((long long)in[(size_t)(16 * jj + i) * 256]);
            cols_inv_regs<S>(ar, v, tw, tw + N, buf[limb], c, jj);
#pragma unroll
            for (int i = 0; i < 16; i++) r[limb][i] = ar.canon(down(ar, v[i]) + ar.load(c0[(size_t)R::row(jj, i) * 256]));
        }
    }
    double m[16];
#pragma unroll
    for (int i = 0; i < 16; i++) m[i] = use > 1 ? crt_centred(r[0][i], r[1][i], crt) : r[0][i] > crt.q0 / 2 ? -(double)(crt.q0 - r[0][i]) : (double)r[0][i];
    __syncthreads();  // the tiles have been read
    // values i and i + 8 are the coefficients t and t + N/2: the first pass multiplies each by its power, the second adds them
#pragma unroll
    for (int i = 0; i < 8; i++) {
        const int row = R::row(jj, i);
        const u32 t = row * 256 + (u32)col;
        const double2 zero = make_double2(0.0, 0.0);
        double2 unread, p0, p1, sum;
        fft_butterfly(make_double2(m[i], 0.0), zero, cos_tab[t], sine<NI>(cos_tab, t), unread, p0);
        fft_butterfly(make_double2(m[i + 8], 0.0), zero, cos_tab[t + NI / 2], sine<NI>(cos_tab, t + NI / 2), unread, p1);
        fft_butterfly(p0, p1, 0.0, 0.0, sum, unread);
        buf[0][row * R::COLS + c] = sum;
    }
    const double2 *x = lds_passes<NI, R2, 1024>(buf[0], buf[1], cos_tab, tid, [&](int cc) { return 4 * (blockIdx.x * R::COLS + cc); });
#pragma unroll
    for (int k = 0; k < 8; k++) {
        const int w = tid + CL_THREADS * k, cc = blockIdx.x * R::COLS + w % R::COLS, k1 = w / R::COLS;
        f[((size_t)blockIdx.y * R2 + k1) * 256 + cc] = x[w];
    }
}
// grid (R2 / 8, n): eight rows k1; out: [n][n_slots], slots slot_begin .. slot_begin + n_slots - 1
template <int S>
__global__ __launch_bounds__(CL_THREADS) void k_cl_dec_rows(const double2 *f, const u32 *slot_of_k, int slot_begin, int n_slots, double inv_scale,
                                                            const double *cos_tab, double *out) {
    constexpr int N = Ring<S>::N, R2 = N / 512;
    __shared__ double2 buf[2][2048];
    const int tid = threadIdx.x;
#pragma unroll
    for (int row = 0; row < 8; row++) buf[0][tid * 8 + row] = f[((size_t)blockIdx.y * R2 + blockIdx.x * 8 + row) * 256 + tid];
    const double2 *x = lds_passes<N, 256, 4 * R2>(buf[0], buf[1], cos_tab, tid, [](int) { return 0; });
#pragma unroll
    for (int m = 0; m < 8; m++) {
        const int w = tid + CL_THREADS * m, row = w & 7, k2 = w >> 3;
        const int j = (int)slot_of_k[blockIdx.x * 8 + row + R2 * k2] - slot_begin;
        if (j >= 0 && j < n_slots) out[(size_t)blockIdx.y * n_slots + j] = x[w].x * inv_scale;
    }
}

// ------------------------------------------------------------------ launchers
void launch_cl_encode(ensi_ctx *ctx, const double *d_slots, int n_pt, int n_slots, int slot0, int slot_step, int y0, double scale, int limbs, double2 *ws,
                      u64 *out, hipStream_t st) {
    ring_dispatch(ctx->log_n, [&](auto s) {
        constexpr int S = decltype(s)::value;
        hipLaunchKernelGGL((k_cl_enc_rows<S>), dim3(ctx->N / 4096, n_pt), dim3(CL_THREADS), 0, st, d_slots, n_slots, slot0, slot_step, y0, ctx->d_slot_of_k,
                           ctx->d_cos, ws);
        hipLaunchKernelGGL((k_cl_enc_cols<S>), dim3(Ring<S>::TILES, n_pt), dim3(CL_THREADS), 0, st, ws, 2.0 * scale / ctx->N, limbs, ctx->d_pc, ctx->d_cos, out);
    });
}

template <int S, int POLYS>
static void launch_rows_key(ensi_ctx *ctx, const u64 *in, const u64 *key, int key_limbs, int limbs, int n, u64 *out, hipStream_t st) {
    const unsigned tiles = (4u * Ring<S>::TILES * limbs + 7) / 8 * 8;
    hipLaunchKernelGGL((k_cl_rows_key<S, POLYS>), dim3(tiles * n), dim3(64), 0, st, in, key, key_limbs, limbs, (u32)n, ctx->d_pc, ctx->d_tw, out);
}

void launch_cl_encrypt_mask(ensi_ctx *ctx, const u64 *d_pk, const int8_t *d_mask, int n, int limbs, u64 *ws, u64 *ct, hipStream_t st) {
    ring_dispatch(ctx->log_n, [&](auto s) {
        constexpr int S = decltype(s)::value, TILES = Ring<S>::TILES;
        hipLaunchKernelGGL((k_cl_fcols_small<S>), dim3(TILES, limbs, n), dim3(CL_THREADS), 0, st, d_mask, ctx->d_pc, ctx->d_tw, ws);
        launch_rows_key<S, 2>(ctx, ws, d_pk, ctx->L, limbs, n, ct, st);
    });
}
void launch_cl_encrypt_add(ensi_ctx *ctx, const int8_t *d_errors, const u64 *pt, int n, int limbs, u64 *ct, hipStream_t st) {
    ring_dispatch(ctx->log_n, [&](auto s) {
        constexpr int S = decltype(s)::value;
        hipLaunchKernelGGL((k_cl_icols_add<S>), dim3(Ring<S>::TILES, 2 * limbs, n), dim3(CL_THREADS), 0, st, ct, d_errors, (size_t)n * ctx->N, pt, limbs, ctx->d_pc,
                           ctx->d_tw);
    });
}

void launch_cl_decrypt(ensi_ctx *ctx, const u64 *d_s_hat, const u64 *ct, int n, int limbs_alloc, int use, const CrtPair &crt, int slot_begin, int n_slots,
                       double inv_scale, u64 *ws, double2 *f, double *out, hipStream_t st) {
    ring_dispatch(ctx->log_n, [&](auto s) {
        constexpr int S = decltype(s)::value, TILES = Ring<S>::TILES;
        hipLaunchKernelGGL((k_cl_fcols_c1<S>), dim3(TILES, use, n), dim3(CL_THREADS), 0, st, ct, limbs_alloc, ctx->d_pc, ctx->d_tw, ws);
        launch_rows_key<S, 1>(ctx, ws, d_s_hat, ctx->L + ctx->K, use, n, ws, st);
        hipLaunchKernelGGL((k_cl_dec_cols<S>), dim3(TILES, n), dim3(CL_THREADS), 0, st, ws, use, ct, limbs_alloc, crt, ctx->d_pc, ctx->d_tw, ctx->d_cos, f);
        hipLaunchKernelGGL((k_cl_dec_rows<S>), dim3(ctx->N / 4096, n), dim3(CL_THREADS), 0, st, f, ctx->d_slot_of_k, slot_begin, n_slots, inv_scale, ctx->d_cos, out);
    });
}
