// Key-switch keys in the format of the fused kernels, and the dispatch to the kernels of a ring (keyswitch16_kernels.h).
#include "common.h"
#include "ntt16_core.h"

template <int S>
void ks16_raise(ensi_ctx *ctx, const Ks16Const &kc, const u64 *ct_base, size_t ct_stride_words, int limb_stride, int n_ct, u64 *dig, bool rows, hipStream_t st);
template <int S>
void ks16_switch(ensi_ctx *ctx, const Ks16Const &kc, const RotDesc *d_desc, int n_rot, u64 *u, int limb_stride_out, bool raw, hipStream_t st, int members);

// ---------------------------------------------------------------- key format
// In place on one key [beta][2][L+K][N] that holds Montgomery residues in position order: into register order, limbs of
// primes below 2^50 as doubles in [0,p), PRIME_WIDE limbs as split centred residues.  A wave owns the 1024 words of four
// rows.  grid (N/1024, L+K, 2*beta)
__global__ __launch_bounds__(64) void k_ks16_key_format(u64 *key, const PrimeConst *pcs, int ext_full, int N) {
    const int lane = threadIdx.x, prime = blockIdx.y;
    const PrimeConst pc = load_prime(pcs, prime);
    u64 *t = key + ((size_t)blockIdx.z * ext_full + prime) * N + (size_t)blockIdx.x * 1024;
    u64 w[16];
#pragma unroll
    for (int i = 0; i < 16; i++) w[i] = t[16 * lane + i];
#pragma unroll
    for (int i = 0; i < 16; i++) {
        acc128 m = {w[i], 0};
        const u64 k = mont_reduce(m, pc.q, pc.qneg_inv);
        if (pc.kind == PRIME_FP) {
            w[i] = (u64)__double_as_longlong((double)k);
        } else if (pc.kind == PRIME_WIDE) {
            const int64_t c = (k > pc.q / 2 ? (int64_t)k - (int64_t)pc.q : (int64_t)k) + (1 << 29);
            w[i] = ((u64)(u32)(u64)(c >> 30) << 32) | (u32)(((u32)c & 0x3fffffffu) - (1u << 29));
        }
    }
    __syncthreads();  // every word of the tile has been read
#pragma unroll
    for (int i = 0; i < 16; i++) t[64 * i + lane] = w[i];
}
// The way back, to ordinary residues in position order.  grid (N/1024, n_rows): row r is limb r % ext_full
__global__ __launch_bounds__(64) void k_ks16_key_plain(u64 *key, const PrimeConst *pcs, int ext_full, int N) {
    const int lane = threadIdx.x;
    const PrimeConst pc = pcs[blockIdx.y % ext_full];
    u64 *t = key + (size_t)blockIdx.y * N + (size_t)blockIdx.x * 1024;
    u64 w[16];
#pragma unroll
    for (int i = 0; i < 16; i++) w[i] = t[64 * i + lane];
#pragma unroll
    for (int i = 0; i < 16; i++) {
        if (pc.kind == PRIME_FP) {
            w[i] = (u64)__longlong_as_double((long long)w[i]);
        } else if (pc.kind == PRIME_WIDE) {
            const int64_t v = (int64_t)(int32_t)(u32)(w[i] >> 32) * (1 << 30) + (int32_t)(u32)w[i];
            w[i] = v < 0 ? (u64)(v + (int64_t)pc.q) : (u64)v;
        } else {
            acc128 m = {w[i], 0};
            w[i] = mont_reduce(m, pc.q, pc.qneg_inv);
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; i++) t[16 * lane + i] = w[i];
}

void launch_ks16_key_format(ensi_ctx *ctx, u64 *key, int beta_full, hipStream_t st) {
    dim3 grid(ctx->N / 1024, ctx->L + ctx->K, 2 * beta_full);
    hipLaunchKernelGGL(k_ks16_key_format, grid, dim3(64), 0, st, key, ctx->d_pc, ctx->L + ctx->K, ctx->N);
}
void launch_ks16_key_plain(ensi_ctx *ctx, u64 *key, int n_rows, hipStream_t st) {
    hipLaunchKernelGGL(k_ks16_key_plain, dim3(ctx->N / 1024, n_rows), dim3(64), 0, st, key, ctx->d_pc, ctx->L + ctx->K, ctx->N);
}


void launch_ks16_raise(ensi_ctx *ctx, const Ks16Const &kc, const u64 *ct_base, size_t ct_stride_words, int limb_stride, int n_ct, u64 *dig, bool rows,
                       hipStream_t st) {
    ring_dispatch(ctx->log_n, [&](auto s) { ks16_raise<decltype(s)::value>(ctx, kc, ct_base, ct_stride_words, limb_stride, n_ct, dig, rows, st); });
}

void launch_ks16_switch(ensi_ctx *ctx, const Ks16Const &kc, const RotDesc *d_desc, int n_rot, u64 *u, int limb_stride_out, bool raw, hipStream_t st,
                        int members) {
    ring_dispatch(ctx->log_n, [&](auto s) { ks16_switch<decltype(s)::value>(ctx, kc, d_desc, n_rot, u, limb_stride_out, raw, st, members); });
}
