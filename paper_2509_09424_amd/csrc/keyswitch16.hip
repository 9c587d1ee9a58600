// Key-switch keys in the format of the fused kernels, and the dispatch to the kernels of a ring (keyswitch16_kernels.h).
#include "api_util.h"
#include "common.h"
#include "ntt16_core.h"

template <int S>
void ks16_raise(ensi_ctx *ctx, const Ks16Const &kc, const u64 *ct_base, size_t ct_stride_words, int limb_stride, int n_ct, u64 *dig, bool rows, hipStream_t st);
template <int S>
void ks16_switch(ensi_ctx *ctx, const Ks16Const &kc, const RotDesc *d_desc, int n_rot, u64 *u, int limb_stride_out, bool raw, hipStream_t st, int members);

// ---------------------------------------------------------------- key format
// Residues in position order -> register order at the source positions of the element g (RowMap), limbs of primes below 2^50
// as centred doubles, PRIME_WIDE limbs as split centred residues, others as Montgomery residues.  Row y of the two arrays is limb y % ext_full.
// A wave writes the 1024 words of four source rows; it reads the four rows they map to.  grid (N/1024, rows)
template <int S>
__global__ __launch_bounds__(64) void k_ks16_key_format(const u64 *in, u64 *out, const PrimeConst *pcs, int ext_full, u32 g, u32 g_inv) {
    typedef RowMap<S> M;
    const int lane = threadIdx.x, rho = lane >> 4, j = lane & 15;
    const PrimeConst pc = load_prime(pcs, blockIdx.y % ext_full);
    const u32 r = M::row(g_inv * M::exponent(blockIdx.x * 4 + rho)), carry = M::carry(r, g);
    const u64 *src = in + (size_t)blockIdx.y * Ring<S>::N + (size_t)r * 256;
    u64 *dst = out + (size_t)blockIdx.y * Ring<S>::N + (size_t)blockIdx.x * 1024;
#pragma unroll
    for (int i = 0; i < 16; i++) {
        u64 w = src[brev8((brev8(16 * j + i) - carry) * g_inv & 255)];
        if (pc.kind == PRIME_FP) {
            w = (u64)__double_as_longlong(w > pc.q / 2 ? (double)w - (double)pc.q : (double)w);
        } else if (pc.kind == PRIME_WIDE) {
            const int64_t c = (w > pc.q / 2 ? (int64_t)w - (int64_t)pc.q : (int64_t)w) + (1 << 29);
            w = ((u64)(u32)(u64)(c >> 30) << 32) | (u32)(((u32)c & 0x3fffffffu) - (1u << 29));
        } else {
            w = mont_mul(w, pc.r2, pc.q, pc.qneg_inv);
        }
        dst[reg_pos(i, lane)] = w;
    }
}
// The way back, to ordinary residues in position order.
template <int S>
__global__ __launch_bounds__(64) void k_ks16_key_plain(const u64 *in, u64 *out, const PrimeConst *pcs, int ext_full, u32 g, u32 g_inv) {
    typedef RowMap<S> M;
    const int lane = threadIdx.x, rho = lane >> 4, j = lane & 15;
    const PrimeConst pc = load_prime(pcs, blockIdx.y % ext_full);
    const u32 r = M::row(g_inv * M::exponent(blockIdx.x * 4 + rho)), carry = M::carry(r, g);
    const u64 *src = in + (size_t)blockIdx.y * Ring<S>::N + (size_t)blockIdx.x * 1024;
    u64 *dst = out + (size_t)blockIdx.y * Ring<S>::N + (size_t)r * 256;
#pragma unroll
    for (int i = 0; i < 16; i++) {
        u64 w = src[reg_pos(i, lane)];
        if (pc.kind == PRIME_FP) {
            const double v = __longlong_as_double((long long)w);
            w = (u64)(v < 0.0 ? v + (double)pc.q : v);
        } else if (pc.kind == PRIME_WIDE) {
            const int64_t v = (int64_t)(int32_t)(u32)(w >> 32) * (1 << 30) + (int32_t)(u32)w;
            w = v < 0 ? (u64)(v + (int64_t)pc.q) : (u64)v;
        } else {
            acc128 m = {w, 0};
            w = mont_reduce(m, pc.q, pc.qneg_inv);
        }
        dst[brev8((brev8(16 * j + i) - carry) * g_inv & 255)] = w;
    }
}

void launch_ks16_key_format(ensi_ctx *ctx, const u64 *in, u64 *out, int n_rows, u32 g, hipStream_t st) {
    ring_dispatch(ctx->log_n, [&](auto s) {
        hipLaunchKernelGGL((k_ks16_key_format<decltype(s)::value>), dim3(ctx->N / 1024, n_rows), dim3(64), 0, st, in, out, ctx->d_pc, ctx->L + ctx->K, g,
                           inv_mod_2n(g, ctx->N));
    });
}
void launch_ks16_key_plain(ensi_ctx *ctx, const u64 *in, u64 *out, int n_rows, u32 g, hipStream_t st) {
    ring_dispatch(ctx->log_n, [&](auto s) {
        hipLaunchKernelGGL((k_ks16_key_plain<decltype(s)::value>), dim3(ctx->N / 1024, n_rows), dim3(64), 0, st, in, out, ctx->d_pc, ctx->L + ctx->K, g,
                           inv_mod_2n(g, ctx->N));
    });
}

void launch_ks16_raise(ensi_ctx *ctx, const Ks16Const &kc, const u64 *ct_base, size_t ct_stride_words, int limb_stride, int n_ct, u64 *dig, bool rows,
                       hipStream_t st) {
    ring_dispatch(ctx->log_n, [&](auto s) { ks16_raise<decltype(s)::value>(ctx, kc, ct_base, ct_stride_words, limb_stride, n_ct, dig, rows, st); });
}

void launch_ks16_switch(ensi_ctx *ctx, const Ks16Const &kc, const RotDesc *d_desc, int n_rot, u64 *u, int limb_stride_out, bool raw, hipStream_t st,
                        int members) {
    ring_dispatch(ctx->log_n, [&](auto s) { ks16_switch<decltype(s)::value>(ctx, kc, d_desc, n_rot, u, limb_stride_out, raw, st, members); });
}
