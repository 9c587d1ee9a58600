// Plaintext multiplication (paper, Preliminaries: Multiplication, PMult) of many ciphertexts, summed per
// output and rescaled once:  out_o = Rescale( sum_{t in terms(o)} src_t (x) pt_t ).  This is the shape of the
// secure RoPE protocol (Alg. 2: three products per output) and of the mask-and-add merge of block-placed
// outputs (c_tot products per output).
//
// A product in R_Q is a pointwise product in the transform domain, so per output limb the work is: forward
// transform of every source limb, multiply by the (pre-transformed) plaintext limb and add, one inverse
// transform, then the rescale across limbs.  Two implementations:
//
//   generic  any ring size and prime: gather the sources, the library's transform, a Montgomery
//            multiply-add kernel, the inverse transform, the integer or fp64 rescale kernel, a strided copy.
//   pm16     N = 2^12 .. 2^16 with ciphertext primes below 2^50, four kernels that keep every intermediate in the
//            layout and number format (exact integers in doubles) of the transform passes around it:
//              k_pm16_fcols            forward column pass of every source limb, read straight from the
//                                      source ciphertexts
//              k_pm16_rows_mac         per output limb and four rows: forward row pass of each term in
//                                      registers, multiply by the plaintext (stored in the register order
//                                      of that pass, so its loads are contiguous), accumulate, and run the
//                                      inverse row pass on the sum -- the products never reach memory
//              (k_pm16_rows, k_pm16_mac  the same in three kernels, where sources enter several products each)
//              k_pm16_icols_last       inverse column pass of the limb the rescale drops, left as the
//                                      centred residue [c_l]
//              k_pm16_icols_rescale    inverse column pass of every other limb fused with
//                                      (c_i - [c_l]) q_l^{-1} mod q_i, written to the output ciphertext
// Both produce canonical residues and agree word for word.
#include "common.h"
#include "ntt16_core.h"

#define PM_THREADS 256

__device__ __forceinline__ double pm_f64(u64 x) { return __longlong_as_double((long long)x); }
__device__ __forceinline__ u64 pm_u64(double x) { return (u64)__double_as_longlong(x); }
// two neighbouring words, 16 bytes to a lane
__device__ __forceinline__ void ld_two(const u64 *base, u32 bytes, double *d) {
    const word_pair p = *(const word_pair *)((const char *)base + bytes);
    d[0] = pm_f64(p[0]);
    d[1] = pm_f64(p[1]);
}
__device__ __forceinline__ void st_two(u64 *base, u32 bytes, double x, double y) { *(word_pair *)((char *)base + bytes) = word_pair{pm_u64(x), pm_u64(y)}; }

// ===================================================================== generic path
// grid (ceil(N/256), 2*l1, n_src): ws_a[slot][c*l1+i][N] <- limb i of component c of the group's distinct source `slot`
__global__ __launch_bounds__(PM_THREADS) void k_pm_gather(PmGroup g, int N) {
    const int idx = blockIdx.x * PM_THREADS + threadIdx.x;
    if (idx >= N) return;
    const int y = blockIdx.y, c = y / g.l1, i = y - c * g.l1, t = blockIdx.z;
    const u64 *src = g.terms[g.owner[t]].src + ((size_t)c * g.limb_stride_in + i) * N;
    g.ws_a[((size_t)t * 2 * g.l1 + y) * N + idx] = src[idx];
}

// grid (ceil(N/256), 2*l1, n_out): ws_b[o][y][N] <- sum_t ws_a[t][y] * pt[t][i]  (transform domain)
__global__ __launch_bounds__(PM_THREADS) void k_pm_mac(PmGroup g, int N, const PrimeConst *pcs) {
    const int idx = blockIdx.x * PM_THREADS + threadIdx.x;
    if (idx >= N) return;
    const int y = blockIdx.y, i = y % g.l1, o = blockIdx.z;
    const u64 q = pcs[i].q, qn = pcs[i].qneg_inv;
    const int t0 = g.begin[o], t1 = g.begin[o + 1];
    u64 acc = 0;
    for (int t = t0; t < t1; t++) {
        const u64 a = g.ws_a[((size_t)g.terms[t].slot * 2 * g.l1 + y) * N + idx];
        const u64 b = g.pt[((size_t)g.terms[t].pt * g.pt_limbs + i) * N + idx];
        acc = add_mod(acc, mont_mul(a, b, q, qn), q);
    }
    g.ws_b[((size_t)o * 2 * g.l1 + y) * N + idx] = acc;
}

// grid (ceil(N/256), 2*(l1-1), n_out): the rescaled limbs of ws_b (limb stride l1) to the output ciphertexts
__global__ __launch_bounds__(PM_THREADS) void k_pm_scatter(PmGroup g, int N) {
    const int idx = blockIdx.x * PM_THREADS + threadIdx.x;
    if (idx >= N) return;
    const int lo = g.l1 - 1;
    const int y = blockIdx.y, c = y / lo, i = y - c * lo, o = blockIdx.z;
    g.out[(size_t)o * g.out_stride + ((size_t)c * g.limb_stride_out + i) * N + idx] = g.ws_b[((size_t)o * 2 * g.l1 + c * g.l1 + i) * N + idx];
}

static LimbMap pm_map(int l1) {
    LimbMap m;
    m.n = l1;
    for (int e = 0; e < ENSI_MAX_EXT; e++) m.prime[e] = e < l1 ? e : 0;
    return m;
}

// d_consts / d_fconsts: the rescale constants with the scalar set to one
void launch_pm_generic(ensi_ctx *ctx, const PmGroup &g, const u64 *d_consts, const double *d_fconsts, hipStream_t st) {
    const int N = ctx->N, nb = (N + PM_THREADS - 1) / PM_THREADS;
    const LimbMap map = pm_map(g.l1);
    if (g.n_src > 0) {
        ScopedTimer t(ctx, "pm_gather", st);
        hipLaunchKernelGGL(k_pm_gather, dim3(nb, 2 * g.l1, g.n_src), dim3(PM_THREADS), 0, st, g, N);
    }
    if (g.n_src > 0) launch_ntt(ctx, g.ws_a, g.n_src * 2 * g.l1, map, false, st);
    {
        ScopedTimer t(ctx, "pm_mac", st);
        hipLaunchKernelGGL(k_pm_mac, dim3(nb, 2 * g.l1, g.n_out), dim3(PM_THREADS), 0, st, g, N, ctx->d_pc);
    }
    launch_ntt(ctx, g.ws_b, g.n_out * 2 * g.l1, map, true, st);
    launch_rescale(ctx, g.ws_b, g.n_out, g.l1, g.l1, d_consts, d_fconsts, st);
    {
        ScopedTimer t(ctx, "pm_scatter", st);
        hipLaunchKernelGGL(k_pm_scatter, dim3(nb, 2 * (g.l1 - 1), g.n_out), dim3(PM_THREADS), 0, st, g, N);
    }
}

// ===================================================================== N = 2^12 .. 2^16, fp64 arithmetic
// Plaintext in the order a wave holds it in the row pass: within the four rows b, lane (rho, j) owns, as its i-th
// value, position 16 j + i of row rho; that value is stored at b*1024 + reg_pos(i, lane), as a double.
// grid (N / 1024, n_rows)
__global__ __launch_bounds__(64) void k_pm16_pt_format(const u64 *in, u64 *out, int N) {
    const int tid = threadIdx.x, rho = tid >> 4, j = tid & 15;
    const size_t base = (size_t)blockIdx.y * N + (size_t)blockIdx.x * 1024;
#pragma unroll
    for (int i = 0; i < 16; i += 2)
        *(word_pair *)(out + base + reg_pos(i, tid)) = word_pair{pm_u64((double)in[base + rho * 256 + 16 * j + i]), pm_u64((double)in[base + rho * 256 + 16 * j + i + 1])};
}
void launch_pm16_pt_format(ensi_ctx *ctx, const u64 *ntt_form, int n_rows, u64 *out, hipStream_t st) {
    hipLaunchKernelGGL(k_pm16_pt_format, dim3(ctx->N / 1024, n_rows), dim3(64), 0, st, ntt_form, out, ctx->N);
}

// grid (TILES, 2*l1, n_src)
template <int S>
__global__ __launch_bounds__(PM_THREADS) void k_pm16_fcols(PmGroup g, const PrimeConst *pcs, const u64 *tw_all) {
    typedef Ring<S> R;
    constexpr size_t PM_N = R::N;
    __shared__ u64 lds[4096];
    const int tid = threadIdx.x, c16 = R::col(tid), jj = R::grp(tid);
    const int y = blockIdx.y, c = y / g.l1, i = y - c * g.l1, t = blockIdx.z;
    const size_t col = (size_t)blockIdx.x * R::COLS + c16;
    auto src = as_global(g.terms[g.owner[t]].src) + ((size_t)c * g.limb_stride_in + i) * PM_N + col;
    u64 *out = g.ws_a + ((size_t)t * 2 * g.l1 + y) * PM_N + col;
    ArithFp ar;
    ar.init(load_prime(pcs, i));
    const u64 *tw = tw_all + (size_t)i * 4 * PM_N;
    double v[16];
#pragma unroll
    for (int k = 0; k < 16; k++) v[k] = ar.load(src[(size_t)R::row(jj, k) * 256]);
    cols_fwd_regs<S>(ar, v, tw, tw + PM_N, lds, c16, jj);
#pragma unroll
    for (int k = 0; k < 16; k++) out[(size_t)(16 * jj + k) * 256] = ar.store_ws_cols(v[k]);
}

// Row passes and products where (nearly) every source enters one product.  A wave takes four rows of one limb of one
// polynomial of one output: per term the forward row pass, times the plaintext, accumulated; then the inverse row pass of
// the sum.  The next operand is requested while the current one is transformed; waves do not wait for each other (with
// blocks of 16 rows and two barriers per term this kernel reached 2.2 TB/s of operand reads).  The two polynomials of an
// output, and then the other outputs, which multiply by the same plaintext tiles, run next to each other on one XCD and
// share those tiles in its L2.  grid (8 * ceil(4 TILES * l1 / 8) * 2 n_out)
template <int S>
__global__ __launch_bounds__(64, 2) void k_pm16_rows_mac(PmGroup g, const PrimeConst *pcs, const u64 *tw_all) {
    typedef Ring<S> R;
    constexpr size_t N = R::N;
    __shared__ u64 lds[ROW_LDS];
    __shared__ ulonglong2 tw1[4 * 16];
    const int lane = threadIdx.x, rho = lane >> 4, j = lane & 15;
    const u32 k = blockIdx.x >> 3, po = k % (2 * (u32)g.n_out), q = k / (2 * (u32)g.n_out) * 8 + (blockIdx.x & 7);
    const int tile = q % (4 * R::TILES), limb = q / (4 * R::TILES), p = po & 1, o = po >> 1;
    if (limb >= g.l1) return;
    const u32 r = tile * 4 + rho;
    ArithFp ar;
    ar.init(load_prime(pcs, limb));
    const u64 *twf = tw_all + (size_t)limb * 4 * N, *twi = twf + 2 * N;
    row_table_to_lds(tw1, twf, twf + N, R::ROWS + r, rho, j);
    TwRegs tw2;
    tw2.load(twf, twf + N, N, r, j);
    const ulonglong2 *tab = tw1 + rho * 16;
    const int t0 = as_const(g.begin)[o], t1 = as_const(g.begin)[o + 1];
    double acc[16], nv[16];
#pragma unroll
    for (int i = 0; i < 16; i++) acc[i] = 0.0;
    const size_t term = (size_t)2 * g.l1 * N, at = (size_t)(p * g.l1 + limb) * N + (size_t)tile * 1024;  // words per source; place in it
    const u64 *a = g.ws_a + at, *b = g.pt + (size_t)limb * N + (size_t)tile * 1024;
    const u32 a_off = (rho * 256 + j) * 8, b_off = reg_pos(0, lane) * 8;
    auto slot_and_pt = [&](int t) { return as_const((const u64 *)(g.terms + t))[1]; };
    if (t0 < t1) {
        const u64 *s = a + (slot_and_pt(t0) >> 32) * term;
#pragma unroll
        for (int i = 0; i < 16; i++) nv[i] = pm_f64(ld_off(s + 16 * i, a_off));
    }
    wave_lds_fence();
#pragma unroll 1
    for (int t = t0; t < t1; t++) {
        const u64 *w_src = b + (size_t)(u32)slot_and_pt(t) * g.pt_limbs * N;
        double v[16], w[16];
#pragma unroll
        for (int i = 0; i < 16; i += 2) ld_two(w_src + reg_pos(i, 0), b_off, w + i);
#pragma unroll
        for (int i = 0; i < 16; i++) v[i] = nv[i];
        if (t + 1 < t1) {
            const u64 *s = a + (slot_and_pt(t + 1) >> 32) * term;
#pragma unroll
            for (int i = 0; i < 16; i++) nv[i] = pm_f64(ld_off(s + 16 * i, a_off));
        }
        row_fwd<true>(ar, v, tab, tw2, lds, rho, j);
#pragma unroll
        for (int i = 0; i < 16; i++) acc[i] += ar.mulmod_np(ar.mid(v[i]), w[i]);
        // a product is below 0.7 q in magnitude: eight of them stay exact in a double
        if (((t - t0) & 7) == 7) {
#pragma unroll
            for (int i = 0; i < 16; i++) acc[i] = ar.mid(acc[i]);
        }
    }
    row_table_to_lds(tw1, twi, twi + N, R::ROWS + r, rho, j);
    tw2.load(twi, twi + N, N, r, j);
    wave_lds_fence();
#pragma unroll
    for (int i = 0; i < 16; i++) acc[i] = ar.mid(acc[i]);
    row_inv(ar, acc, tab, tw2, lds, rho, j);
    u64 *out = g.ws_b + (size_t)o * term + at;
#pragma unroll
    for (int i = 0; i < 16; i++) st_off(out + 16 * i, a_off, ar.store_ws_inv(acc[i]));
}

// Where sources enter several products each, their row passes are run once (k_pm16_rows<true>), the products are formed
// on whole tiles (k_pm16_mac) and the sums brought back (k_pm16_rows<false>).  Between these the words of a wave's four rows
// are in register order (reg_pos).
// grid (4 TILES, 2 * l1 * ceil(n / PM_ROWS_GROUP)): a wave takes four rows of polynomial-limb y for up to PM_ROWS_GROUP of the n
// ciphertexts (the twiddles are fetched once), in place.
#define PM_ROWS_GROUP 8
template <int S, bool FWD>
__global__ __launch_bounds__(64, 2) void k_pm16_rows(u64 *data, int n, int l1, const PrimeConst *pcs, const u64 *tw_all) {
    typedef Ring<S> R;
    constexpr size_t N = R::N;
    __shared__ u64 lds[ROW_LDS];
    __shared__ ulonglong2 tw1[4 * 16];
    const int lane = threadIdx.x, rho = lane >> 4, j = lane & 15;
    const int y = blockIdx.y % (2 * l1), c0 = blockIdx.y / (2 * l1) * PM_ROWS_GROUP, limb = y % l1;
    const u32 r = blockIdx.x * 4 + rho;
    ArithFp ar;
    ar.init(load_prime(pcs, limb));
    const u64 *tw = tw_all + (size_t)limb * 4 * N + (FWD ? 0 : 2 * N);
    row_table_to_lds(tw1, tw, tw + N, R::ROWS + r, rho, j);
    TwRegs tw2;
    tw2.load(tw, tw + N, N, r, j);
    const ulonglong2 *tab = tw1 + rho * 16;
    const u32 row_off = (rho * 256 + j) * 8, reg_off = reg_pos(0, lane) * 8;
    const size_t ct = (size_t)2 * l1 * N;
    u64 *g = data + c0 * ct + (size_t)y * N + (size_t)blockIdx.x * 1024;
    const int n_here = min(PM_ROWS_GROUP, n - c0);
    double v[16], nv[16];
    auto fetch = [&](const u64 *src) {
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
            if (FWD) {
                nv[i] = pm_f64(ld_off(src + 16 * i, row_off));
                nv[i + 1] = pm_f64(ld_off(src + 16 * i + 16, row_off));
            } else {
                ld_two(src + reg_pos(i, 0), reg_off, nv + i);
            }
        }
    };
    fetch(g);
    wave_lds_fence();
#pragma unroll 1
    for (int c = 0; c < n_here; c++) {
#pragma unroll
        for (int i = 0; i < 16; i++) v[i] = nv[i];
        if (c + 1 < n_here) fetch(g + ct);
        if (FWD) row_fwd<true>(ar, v, tab, tw2, lds, rho, j);
        else row_inv(ar, v, tab, tw2, lds, rho, j);
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
            const double x = ar.mid(v[i]), y = ar.mid(v[i + 1]);
            if (FWD) {
                st_two(g + reg_pos(i, 0), reg_off, x, y);
            } else {
                st_off(g + 16 * i, row_off, pm_u64(x));
                st_off(g + 16 * i + 16, row_off, pm_u64(y));
            }
        }
        g += ct;
    }
}

// Sums of products of transformed sources for PM_MAC_OUT outputs at a time: an operand word is read once for them.  All groups
// of outputs of a tile of 1024 words run together on one XCD, whose L2 then serves their sources and plaintexts
// (127 sources and 192 plaintexts are 0.9 MiB a tile).  entries: per group a list of (source, plaintext per output or
// -1); entry_begin: [n_groups + 1].  grid (8 * ceil(N / 1024 * l1 / 8) * n_groups)
template <int S>
__global__ __launch_bounds__(PM_THREADS) void k_pm16_mac(PmGroup g, const PmEntry *entries, const int32_t *entry_begin, int n_groups, const PrimeConst *pcs) {
    typedef Ring<S> R;
    constexpr size_t N = R::N;
    const u32 k = blockIdx.x >> 3, grp = k % (u32)n_groups, q = k / (u32)n_groups * 8 + (blockIdx.x & 7);
    const int tile = q % (4 * R::TILES), limb = q / (4 * R::TILES);
    if (limb >= g.l1) return;
    ArithFp ar;
    ar.init(load_prime(pcs, limb));
    const size_t poly = (size_t)g.l1 * N;
    const u64 *a = g.ws_a + (size_t)limb * N + (size_t)tile * 1024, *b = g.pt + (size_t)limb * N + (size_t)tile * 1024;
    const u32 off = threadIdx.x * 16;  // two words to a load: values i and i + 1 of a thread are neighbours
    double acc[PM_MAC_OUT][2][4];
#pragma unroll
    for (int o = 0; o < PM_MAC_OUT; o++)
#pragma unroll
        for (int i = 0; i < 4; i++) acc[o][0][i] = acc[o][1][i] = 0.0;
    const int e0 = as_const(entry_begin)[grp], e1 = as_const(entry_begin)[grp + 1];
    double x[2][4];
    auto fetch = [&](int slot) {
        const u64 *s = a + (size_t)slot * 2 * poly;
#pragma unroll
        for (int i = 0; i < 4; i += 2) {
            ld_two(s + 256 * i, off, x[0] + i);
            ld_two(s + poly + 256 * i, off, x[1] + i);
        }
    };
    auto entry = [&](int e, int w) { return as_const((const int32_t *)(entries + e))[w]; };
    if (e0 < e1) fetch(entry(e0, 0));
#pragma unroll 1
    for (int e = e0; e < e1; e++) {
        double v[2][4], w[PM_MAC_OUT][4];
#pragma unroll
        for (int o = 0; o < PM_MAC_OUT; o++) {
            const int pt = entry(e, 1 + o);
            if (pt >= 0) {
#pragma unroll
                for (int i = 0; i < 4; i += 2) ld_two(b + (size_t)pt * g.pt_limbs * N + 256 * i, off, w[o] + i);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; i++) {
            v[0][i] = x[0][i];
            v[1][i] = x[1][i];
        }
        if (e + 1 < e1) fetch(entry(e + 1, 0));
#pragma unroll
        for (int o = 0; o < PM_MAC_OUT; o++) {
            if (entry(e, 1 + o) >= 0) {
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    acc[o][0][i] += ar.mulmod_np(v[0][i], w[o][i]);
                    acc[o][1][i] += ar.mulmod_np(v[1][i], w[o][i]);
                }
            }
        }
        // a product is below 0.7 q in magnitude: eight of them stay exact in a double
        if (((e - e0) & 7) == 7) {
#pragma unroll
            for (int o = 0; o < PM_MAC_OUT; o++)
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    acc[o][0][i] = ar.mid(acc[o][0][i]);
                    acc[o][1][i] = ar.mid(acc[o][1][i]);
                }
        }
    }
#pragma unroll
    for (int o = 0; o < PM_MAC_OUT; o++) {
        const u32 out_idx = grp * PM_MAC_OUT + o;
        if (out_idx < (u32)g.n_out) {
            u64 *d = g.ws_b + (size_t)out_idx * 2 * poly + (size_t)limb * N + (size_t)tile * 1024;
#pragma unroll
            for (int i = 0; i < 4; i += 2) {
                st_two(d + 256 * i, off, ar.mid(acc[o][0][i]), ar.mid(acc[o][0][i + 1]));
                st_two(d + poly + 256 * i, off, ar.mid(acc[o][1][i]), ar.mid(acc[o][1][i + 1]));
            }
        }
    }
}

// grid (TILES, 2, n_out): ws_last[o][c][N] <- centred residue of limb l1-1 (coefficient form)
template <int S>
__global__ __launch_bounds__(PM_THREADS) void k_pm16_icols_last(PmGroup g, const PrimeConst *pcs, const u64 *tw_all) {
    typedef Ring<S> R;
    constexpr size_t PM_N = R::N;
    __shared__ u64 lds[4096];
    const int tid = threadIdx.x, c16 = R::col(tid), jj = R::grp(tid);
    const int c = blockIdx.y, o = blockIdx.z, i = g.l1 - 1;
    const size_t col = (size_t)blockIdx.x * R::COLS + c16;
    const u64 *src = g.ws_b + ((size_t)o * 2 * g.l1 + c * g.l1 + i) * PM_N + col;
    u64 *dst = g.ws_last + ((size_t)o * 2 + c) * PM_N + col;
    ArithFp ar;
    ar.init(load_prime(pcs, i));
    const u64 *tw = tw_all + (size_t)i * 4 * PM_N + 2 * PM_N;
    double v[16];
#pragma unroll
    for (int k = 0; k < 16; k++) v[k] = pm_f64(src[(size_t)(16 * jj + k) * 256]);
    cols_inv_regs<S>(ar, v, tw, tw + PM_N, lds, c16, jj);
#pragma unroll
    for (int k = 0; k < 16; k++) dst[(size_t)R::row(jj, k) * 256] = pm_u64(ar.mid(ar.mulmod(v[k], ar.ninv, ar.ninv_p)));
}

// grid (TILES, 2*(l1-1), n_out)
template <int S>
__global__ __launch_bounds__(PM_THREADS) void k_pm16_icols_rescale(PmGroup g, PmRescale rs, const PrimeConst *pcs, const u64 *tw_all) {
    typedef Ring<S> R;
    constexpr size_t PM_N = R::N;
    __shared__ u64 lds[4096];
    const int tid = threadIdx.x, c16 = R::col(tid), jj = R::grp(tid);
    const int lo = g.l1 - 1;
    const int y = blockIdx.y, c = y / lo, i = y - c * lo, o = blockIdx.z;
    const size_t col = (size_t)blockIdx.x * R::COLS + c16;
    const u64 *src = g.ws_b + ((size_t)o * 2 * g.l1 + c * g.l1 + i) * PM_N + col;
    const u64 *last = g.ws_last + ((size_t)o * 2 + c) * PM_N + col;
    u64 *dst = g.out + (size_t)o * g.out_stride + ((size_t)c * g.limb_stride_out + i) * PM_N + col;
    ArithFp ar;
    ar.init(load_prime(pcs, i));
    const u64 *tw = tw_all + (size_t)i * 4 * PM_N + 2 * PM_N;
    const double w = rs.w[i], wp = rs.wp[i];
    double v[16], tl[16];
#pragma unroll
    for (int k = 0; k < 16; k++) v[k] = pm_f64(src[(size_t)(16 * jj + k) * 256]);
#pragma unroll
    for (int k = 0; k < 16; k++) tl[k] = pm_f64(last[(size_t)R::row(jj, k) * 256]);
    cols_inv_regs<S>(ar, v, tw, tw + PM_N, lds, c16, jj);
#pragma unroll
    for (int k = 0; k < 16; k++) {
        const double x = ar.mid(ar.mulmod(v[k], ar.ninv, ar.ninv_p));
        const double z = ar.mid(x - ar.mid(tl[k]));
        dst[(size_t)R::row(jj, k) * 256] = ar.canon(ar.mulmod(z, w, wp));
    }
}

void launch_pm16(ensi_ctx *ctx, const PmGroup &g, const PmRescale &rs, hipStream_t st) {
    ring_dispatch(ctx->log_n, [&](auto s) {
        constexpr int S = decltype(s)::value, TILES = Ring<S>::TILES;
        if (g.n_src > 0) {
            ScopedTimer t(ctx, "pm_fcols", st);
            hipLaunchKernelGGL((k_pm16_fcols<S>), dim3(TILES, 2 * g.l1, g.n_src), dim3(PM_THREADS), 0, st, g, ctx->d_pc, ctx->d_tw);
        }
        const unsigned tiles = (4u * TILES * g.l1 + 7) / 8 * 8;  // tiles of four rows, in groups of eight (one per XCD)
        if (g.entries) {
            const int n_groups = (g.n_out + PM_MAC_OUT - 1) / PM_MAC_OUT;
            {
                ScopedTimer t(ctx, "pm_frows", st);
                hipLaunchKernelGGL((k_pm16_rows<S, true>), dim3(4 * TILES, 2 * g.l1 * ((g.n_src + PM_ROWS_GROUP - 1) / PM_ROWS_GROUP)), dim3(64), 0, st, g.ws_a,
                                   g.n_src, g.l1, ctx->d_pc, ctx->d_tw);
            }
            {
                ScopedTimer t(ctx, "pm_mac", st);
                hipLaunchKernelGGL((k_pm16_mac<S>), dim3(tiles * n_groups), dim3(PM_THREADS), 0, st, g, g.entries, g.entry_begin, n_groups, ctx->d_pc);
            }
            {
                ScopedTimer t(ctx, "pm_irows", st);
                hipLaunchKernelGGL((k_pm16_rows<S, false>), dim3(4 * TILES, 2 * g.l1 * ((g.n_out + PM_ROWS_GROUP - 1) / PM_ROWS_GROUP)), dim3(64), 0, st, g.ws_b,
                                   g.n_out, g.l1, ctx->d_pc, ctx->d_tw);
            }
        } else {
            ScopedTimer t(ctx, "pm_rows_mac", st);
            hipLaunchKernelGGL((k_pm16_rows_mac<S>), dim3(tiles * 2 * g.n_out), dim3(64), 0, st, g, ctx->d_pc, ctx->d_tw);
        }
        {
            ScopedTimer t(ctx, "pm_icols_last", st);
            hipLaunchKernelGGL((k_pm16_icols_last<S>), dim3(TILES, 2, g.n_out), dim3(PM_THREADS), 0, st, g, ctx->d_pc, ctx->d_tw);
        }
        {
            ScopedTimer t(ctx, "pm_icols_rescale", st);
            hipLaunchKernelGGL((k_pm16_icols_rescale<S>), dim3(TILES, 2 * (g.l1 - 1), g.n_out), dim3(PM_THREADS), 0, st, g, rs, ctx->d_pc, ctx->d_tw);
        }
    });
}
