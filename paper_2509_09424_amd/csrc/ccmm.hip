// Ciphertext-ciphertext multiplication (paper, Preliminaries: Multiplication, Mult) for the ciphertext-
// ciphertext matrix product of the CCMM section:  out_o = Rescale(Relin(sum_t a_t (x) b_t)).
//
// The tensor product of two ciphertexts is three polynomials (d0, d1, d2) = (a0 b0, a0 b1 + a1 b0, a1 b1),
// products in R_{Q_l}, i.e. pointwise in the transform domain.  The products of one output are added there,
// transformed back once, d2 is key-switched from s^2 to s with the evaluation key (the same raise / inner
// product / ModDown kernels as a rotation, with the identity automorphism, fed (d0, d2) as if it were a
// ciphertext so that d0 is added on the way), d1 is added and the result rescaled.
//
// Kernels here: the gather of the two polynomials of every distinct operand of a group (an operand that enters
// several products is transformed once), the multiply-add that forms
// (d0, d2, d1) per output, the addition of d1 and a strided ciphertext addition (used by the rotate-and-add
// steps of the element replication).  Transforms, key switch, rescale and the final strided copy are the
// library's existing kernels.
#include "common.h"
#include "ntt16_core.h"

#define MM_THREADS 256

// grid (ceil(N/256) * n_ops, 2*l1): ws_a[u][p*l1+i][N] <- polynomial p, limb i of distinct operand u
__global__ __launch_bounds__(MM_THREADS) void k_mm_gather(MmGroup g, int N, int nb) {
    const int u = blockIdx.x / nb;
    const int idx = (blockIdx.x - u * nb) * MM_THREADS + threadIdx.x;
    if (idx >= N) return;
    const int y = blockIdx.y, p = y / g.l1, i = y - p * g.l1;
    const MmOperand op = g.ops[u];
    g.ws_a[((size_t)u * 2 * g.l1 + y) * N + idx] = op.p[((size_t)p * op.limb_stride + i) * N + idx];
}

// grid (ceil(N/256), l1, n_out): ws_d[o][0|1|2][i][N] <- d0, d2, d1 (transform domain).  Operands are ordinary
// residues: a Montgomery product carries a factor 2^-64, removed once per sum with 2^128 mod q.
__global__ __launch_bounds__(MM_THREADS) void k_mm_tensor_mac(MmGroup g, int N, const PrimeConst *pcs) {
    const int idx = blockIdx.x * MM_THREADS + threadIdx.x;
    if (idx >= N) return;
    const int i = blockIdx.y, o = blockIdx.z;
    const PrimeConst pc = pcs[i];
    const u64 q = pc.q, qn = pc.qneg_inv;
    const int t0 = g.begin[o], t1 = g.begin[o + 1];
    u64 d0 = 0, d1 = 0, d2 = 0;
    const size_t poly = (size_t)g.l1 * N;
    for (int t = t0; t < t1; t++) {
        const MmPair pr = g.pairs[t - g.t_base];
        const u64 *xa = g.ops[pr.a].t + (size_t)i * N + idx;
        const u64 *xb = g.ops[pr.b].t + (size_t)i * N + idx;
        const u64 a0 = xa[0], a1 = xa[poly], b0 = xb[0], b1 = xb[poly];
        d0 = add_mod(d0, mont_mul(a0, b0, q, qn), q);
        d1 = add_mod(d1, add_mod(mont_mul(a0, b1, q, qn), mont_mul(a1, b0, q, qn), q), q);
        d2 = add_mod(d2, mont_mul(a1, b1, q, qn), q);
    }
    u64 *out = g.ws_d + ((size_t)o * 3 * g.l1 + i) * N + idx;
    out[0] = mont_mul(d0, pc.r2, q, qn);
    out[poly] = mont_mul(d2, pc.r2, q, qn);
    out[2 * poly] = mont_mul(d1, pc.r2, q, qn);
}

// The same sums for TX x TY outputs at a time, primes below 2^50: output (x, y) of a group adds a_x (x) b_y over the group's
// entries.  Every operand word a block reads enters TY or TX products, and all groups of a range of words run together on one
// XCD, so that operands shared by groups come from its L2: memory is read about once, which is what bounds this kernel (the
// plain kernel reads four operand words per product).
// Arithmetic: words are taken as two 25-bit halves, products of halves added up in 64-bit integers -- four multiply-adds per
// product, against six instructions for a reduced product in fp64 -- and reduced every MM_FOLD entries and at the end.
// The middle polynomial is formed from (a0 + a1)(b0 + b1): twelve multiply-adds instead of sixteen per pair.
// grid (8 * ceil(N / 256 * l1 / 8) * n_groups)
#define MM_FOLD 512  // a sum of 512 middle terms of twice 2^52 stays below 2^62.1
template <int TX, int TY>
__global__ __launch_bounds__(MM_THREADS, TX * TY > 4 ? 2 : 3) void k_mm_mac(MmGroup g, int N, const PrimeConst *pcs) {
    const u32 k = blockIdx.x >> 3, grp = k % (u32)g.n_groups, q = k / (u32)g.n_groups * 8 + (blockIdx.x & 7);
    const int per_limb = N / MM_THREADS, limb = q / per_limb;
    if (limb >= g.l1) return;
    const u32 off = ((q - limb * per_limb) * MM_THREADS + threadIdx.x) * 8;
    const size_t poly = (size_t)g.l1 * N, at = (size_t)limb * N;
    ArithFp ar;
    ar.init(load_prime(pcs, limb));
    // sums of products of halves: [0] low * low, [1] the two mixed ones, [2] high * high; of a0 b0, (a0+a1)(b0+b1), a1 b1
    int64_t s[TX][TY][3][3];
#pragma unroll
    for (int x = 0; x < TX; x++)
#pragma unroll
        for (int y = 0; y < TY; y++)
#pragma unroll
            for (int d = 0; d < 9; d++) s[x][y][d / 3][d % 3] = 0;
    const double c25r = ar.mid(33554432.0), c25 = c25r < 0.0 ? c25r + ar.p : c25r;
    const double c50r = ar.mid(ar.mulmod_np(ar.mid(c25), c25)), c50 = c50r < 0.0 ? c50r + ar.p : c50r;
    auto residue = [&](int64_t v) {  // centred
        const double h = (double)(int)(v >> 32) * 4294967296.0;
        return ar.mid(fma(-rint(h * ar.pinv), ar.p, h) + (double)(u32)v);
    };
    auto reduce = [&](const int64_t *v) { return ar.mid(ar.mulmod_np(residue(v[2]), c50) + ar.mulmod_np(residue(v[1]), c25) + residue(v[0])); };
    const int e0 = as_const(g.entry_begin)[grp], e1 = as_const(g.entry_begin)[grp + 1];
    auto index = [&](int e, int w) { return as_const((const int32_t *)(g.entries + e))[w]; };
    struct Words {
        u64 a[TX][2], b[TY][2];
    };
    auto place_of = [&](int i) { return as_const((const u64 *)(g.ops + i))[1]; };  // MmOperand.t
    auto two = [&](u64 p, u64 *d) {
        const u64 *s0 = (const u64 *)p + at;
        d[0] = *as_global((const u64 *)((const char *)s0 + off));
        d[1] = *as_global((const u64 *)((const char *)(s0 + poly) + off));
    };
    // In a grid of outputs the words of two entries are on their way while one is multiplied, with the places of the next one
    // and the indices of the one after it in scalar registers: there the kernel waited for operand words and for look-ups, not
    // for multiply-adds or memory (96 x 32 x 4 products at 15 limbs: 17.8 ms with one entry ahead, 14.4 so).
    // No load hangs on a branch, so that the compiler can count the loads it does not wait for: an operand that an entry does not
    // name -- only products of outputs that do not exist lack one -- is read from another place.
    u64 pa[TX], pb[TY];
    int ia[TX], ib[TY];
    auto look_up = [&](int e) {
        e = min(e, e1 - 1);
#pragma unroll
        for (int x = 0; x < TX; x++) ia[x] = index(e, x);
#pragma unroll
        for (int y = 0; y < TY; y++) ib[y] = index(e, 4 + y);
    };
    auto place = [&]() {
#pragma unroll
        for (int x = 0; x < TX; x++) pa[x] = place_of(max(ia[x], 0));
#pragma unroll
        for (int y = 0; y < TY; y++) pb[y] = place_of(max(ib[y], 0));
    };
    auto fetch_placed = [&](Words &w, int e) {  // the words of entry e, whose places are at hand
#pragma unroll
        for (int x = 0; x < TX; x++) two(pa[x], w.a[x]);
#pragma unroll
        for (int y = 0; y < TY; y++) two(pb[y], w.b[y]);
        place();
        look_up(e + 2);
    };
    // Without a grid every operand is read about once, at the rate of memory, and one entry ahead is enough.  An entry then names one
    // to four left operands, and those that it does not name are not read: where sums share no right operand that is three of
    // four (four sums of 96 products at 15 limbs: 2.2 ms, and 2.9 with all four read).  Sums that share every right operand: 3.1 ms
    // for 16 GB, 3.25 with two entries ahead.
    auto fetch_named = [&](Words &w, int e) {
        if (e >= e1) return;
#pragma unroll
        for (int x = 0; x < TX; x++) {
            const int i = index(e, x);
            if (i >= 0) two(place_of(i), w.a[x]);
            else w.a[x][0] = w.a[x][1] = 0;
        }
#pragma unroll
        for (int y = 0; y < TY; y++) two(place_of(index(e, 4 + y)), w.b[y]);
    };
    constexpr int AHEAD = TY > 1 ? 2 : 1;
    auto multiply = [&](Words &w, int e) {
        // halves of a0, a0 + a1, a1 (and b alike): at most 26 bits
        int al[TX][3], ah[TX][3], bl[TY][3], bh[TY][3];
        auto halves = [](const u64 *d, int *l, int *h) {
            l[0] = (int)((u32)d[0] & 0x1ffffffu);
            h[0] = (int)(u32)(d[0] >> 25);
            l[2] = (int)((u32)d[1] & 0x1ffffffu);
            h[2] = (int)(u32)(d[1] >> 25);
            l[1] = l[0] + l[2];
            h[1] = h[0] + h[2];
        };
#pragma unroll
        for (int x = 0; x < TX; x++) halves(w.a[x], al[x], ah[x]);
#pragma unroll
        for (int y = 0; y < TY; y++) halves(w.b[y], bl[y], bh[y]);
        if (TY > 1) {
            fetch_placed(w, e + AHEAD);
            __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of the multiply-adds
        } else {
            fetch_named(w, e + AHEAD);
        }
#pragma unroll
        for (int x = 0; x < TX; x++)
#pragma unroll
            for (int y = 0; y < TY; y++)
#pragma unroll
                for (int d = 0; d < 3; d++) {
                    s[x][y][d][0] = mad_i(al[x][d], bl[y][d], s[x][y][d][0]);
                    s[x][y][d][1] = mad_i(al[x][d], bh[y][d], s[x][y][d][1]);
                    s[x][y][d][1] = mad_i(ah[x][d], bl[y][d], s[x][y][d][1]);
                    s[x][y][d][2] = mad_i(ah[x][d], bh[y][d], s[x][y][d][2]);
                }
    };
    Words w0, w1;
    if (TY == 1) {
        fetch_named(w0, e0);
    } else if (e0 < e1) {
        look_up(e0);
        place();
        look_up(e0 + 1);
        fetch_placed(w0, e0);
        fetch_placed(w1, e0 + 1);
    }
#pragma unroll 1
    for (int e = e0; e < e1; e += AHEAD) {
        multiply(w0, e);
        if (AHEAD > 1) {
            if (e + 1 == e1) break;
            multiply(w1, e + 1);
        }
        if ((e - e0) % MM_FOLD == MM_FOLD - AHEAD) {
#pragma unroll
            for (int x = 0; x < TX; x++)
#pragma unroll
                for (int y = 0; y < TY; y++)
#pragma unroll
                    for (int d = 0; d < 3; d++) {
                        s[x][y][d][0] = (int64_t)reduce(s[x][y][d]);
                        s[x][y][d][1] = s[x][y][d][2] = 0;
                    }
        }
    }
#pragma unroll
    for (int x = 0; x < TX; x++)
#pragma unroll
        for (int y = 0; y < TY; y++) {
            const int o = as_const(g.entry_out)[(grp * TX + x) * TY + y];
            if (o < 0) continue;
            const double d0 = reduce(s[x][y][0]), d2 = reduce(s[x][y][2]), d1 = reduce(s[x][y][1]) - d0 - d2;
            u64 *out = g.ws_d + (size_t)o * 3 * poly + at;
            st_off(out, off, ar.canon(d0));
            st_off(out + poly, off, ar.canon(d2));
            st_off(out + 2 * poly, off, ar.canon(d1));
        }
}

// grid (ceil(N/256), l1, n_out): ws_e[o][1][i] += ws_d[o][2][i]  (d1 joins the second polynomial)
__global__ __launch_bounds__(MM_THREADS) void k_mm_add_d1(MmGroup g, int N, const PrimeConst *pcs) {
    const int idx = blockIdx.x * MM_THREADS + threadIdx.x;
    if (idx >= N) return;
    const int i = blockIdx.y, o = blockIdx.z;
    u64 *e = g.ws_e + ((size_t)o * 2 * g.l1 + g.l1 + i) * N + idx;
    *e = add_mod(*e, g.ws_d[((size_t)o * 3 * g.l1 + 2 * g.l1 + i) * N + idx], pcs[i].q);
}

// grid (ceil(N/256), 2*l1, n): a[c][poly][i] += b[c][poly][i] on batches with their own limb strides
__global__ __launch_bounds__(MM_THREADS) void k_ct_add(u64 *a, int stride_a, const u64 *b, int stride_b, int l1, int N, const PrimeConst *pcs) {
    const int idx = blockIdx.x * MM_THREADS + threadIdx.x;
    if (idx >= N) return;
    const int y = blockIdx.y, p = y / l1, i = y - p * l1, c = blockIdx.z;
    u64 *x = a + ((size_t)c * 2 * stride_a + (size_t)p * stride_a + i) * N + idx;
    *x = add_mod(*x, b[((size_t)c * 2 * stride_b + (size_t)p * stride_b + i) * N + idx], pcs[i].q);
}

// grid (ceil(N/256), 2*limbs_out, n_out): the first limbs_out limbs of ws_e (limb stride l1) to the output ciphertexts
__global__ __launch_bounds__(MM_THREADS) void k_mm_scatter(MmGroup g, int N) {
    const int idx = blockIdx.x * MM_THREADS + threadIdx.x;
    if (idx >= N) return;
    const int lo = g.limbs_out;
    const int y = blockIdx.y, c = y / lo, i = y - c * lo, o = blockIdx.z;
    g.out[(size_t)o * g.out_stride + ((size_t)c * g.limb_stride_out + i) * N + idx] = g.ws_e[((size_t)o * 2 * g.l1 + c * g.l1 + i) * N + idx];
}

static LimbMap mm_map(int l1) {
    LimbMap m;
    m.n = l1;
    for (int e = 0; e < ENSI_MAX_EXT; e++) m.prime[e] = e < l1 ? e : 0;
    return m;
}

// gather -> forward transform -> tensor multiply-add -> inverse transform: leaves (d0, d2, d1) of every output of
// the group in ws_d, coefficient form
void launch_mm_tensor(ensi_ctx *ctx, const MmGroup &g, hipStream_t st) {
    const int N = ctx->N, nb = (N + MM_THREADS - 1) / MM_THREADS;
    const LimbMap map = mm_map(g.l1);
    if (g.n_ops > 0) {
        if (ctx->log_n >= 12) {
            // the forward column pass reads the operands where they lie
            launch_ntt16_gather(ctx, g.ws_a, g.ops, g.n_ops, g.l1, st);
        } else {
            {
                ScopedTimer t(ctx, "mm_gather", st);
                hipLaunchKernelGGL(k_mm_gather, dim3((unsigned)nb * g.n_ops, 2 * g.l1), dim3(MM_THREADS), 0, st, g, N, nb);
            }
            launch_ntt(ctx, g.ws_a, g.n_ops * 2 * g.l1, map, false, st);
        }
    }
    {
        ScopedTimer t(ctx, "mm_tensor_mac", st);
        const unsigned blocks = ((unsigned)nb * g.l1 + 7) / 8 * 8 * g.n_groups;
        if (g.n_groups > 0 && g.tile_y == 2)
            hipLaunchKernelGGL((k_mm_mac<4, 2>), dim3(blocks), dim3(MM_THREADS), 0, st, g, N, ctx->d_pc);
        else if (g.n_groups > 0)
            hipLaunchKernelGGL((k_mm_mac<4, 1>), dim3(blocks), dim3(MM_THREADS), 0, st, g, N, ctx->d_pc);
        else
            hipLaunchKernelGGL(k_mm_tensor_mac, dim3(nb, g.l1, g.n_out), dim3(MM_THREADS), 0, st, g, N, ctx->d_pc);
    }
    launch_ntt(ctx, g.ws_d, g.n_out * 3 * g.l1, map, true, st);
}

void launch_mm_add_d1(ensi_ctx *ctx, const MmGroup &g, hipStream_t st) {
    const int N = ctx->N, nb = (N + MM_THREADS - 1) / MM_THREADS;
    ScopedTimer t(ctx, "mm_add_d1", st);
    hipLaunchKernelGGL(k_mm_add_d1, dim3(nb, g.l1, g.n_out), dim3(MM_THREADS), 0, st, g, N, ctx->d_pc);
}

void launch_ct_add(ensi_ctx *ctx, u64 *a, int stride_a, const u64 *b, int stride_b, int l1, int n, hipStream_t st) {
    const int N = ctx->N, nb = (N + MM_THREADS - 1) / MM_THREADS;
    ScopedTimer t(ctx, "ct_add", st);
    hipLaunchKernelGGL(k_ct_add, dim3(nb, 2 * l1, n), dim3(MM_THREADS), 0, st, a, stride_a, b, stride_b, l1, N, ctx->d_pc);
}

void launch_mm_scatter(ensi_ctx *ctx, const MmGroup &g, hipStream_t st) {
    const int N = ctx->N, nb = (N + MM_THREADS - 1) / MM_THREADS;
    ScopedTimer t(ctx, "mm_scatter", st);
    hipLaunchKernelGGL(k_mm_scatter, dim3(nb, 2 * g.limbs_out, g.n_out), dim3(MM_THREADS), 0, st, g, N);
}
