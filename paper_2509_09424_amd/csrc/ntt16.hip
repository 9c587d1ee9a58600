// Negacyclic NTT for the rings N = 2^12 .. 2^16: two passes, each of up to two steps of four stages held in
// registers with one exchange through LDS in between (ntt16_core.h has the cut of the stages and the arithmetic).
//
// Same transform, stage order, twiddle tables (psi^bitrev(k)) and output order as the generic kernels in ntt.hip; both
// write canonical residues, so results are bit-identical.  In a step a thread owns 16 elements whose indices differ
// in the 4 bits the step works on; the twiddle of local stage k and local butterfly group g is
// table[(Mbase << k) + g] with
//   Mbase = 1 | 2^S + jj | ROWS + r | (ROWS + r) * 16 + j
// for column step 1 | column step 2 | row step 1 | row step 2 (jj: the thread's group of 16 rows, r: the row, j: the
// thread's slot of 16 in the row).
#include <algorithm>

#include "common.h"
#include "ntt16_core.h"

#define N16_THREADS 256

// ---- column pass of one tile.  gin: where the forward pass reads it (the same place as g for a transform in place)
template <int S, bool FWD, class A>
__device__ __forceinline__ void cols_body(u64 *g, const u64 *gin, const u64 *tw, const PrimeConst &pc, u64 *lds) {
    typedef Ring<S> R;
    A ar;
    ar.init(pc);
    const int c = R::col(threadIdx.x), jj = R::grp(threadIdx.x);
    typename A::T v[16];
    if (FWD) {
#pragma unroll
        for (int i = 0; i < 16; i++) v[i] = ar.load(gin[(size_t)R::row(jj, i) * 256 + c]);
        cols_fwd_regs<S>(ar, v, tw, tw + R::N, lds, c, jj);
#pragma unroll
        for (int i = 0; i < 16; i++) g[(size_t)(16 * jj + i) * 256 + c] = ar.store_fwd(v[i]);
    } else {
#pragma unroll
        for (int i = 0; i < 16; i++) v[i] = ar.center(ar.load(g[(size_t)(16 * jj + i) * 256 + c]));
        cols_inv_regs<S>(ar, v, tw, tw + R::N, lds, c, jj);
#pragma unroll
        for (int i = 0; i < 16; i++) g[(size_t)R::row(jj, i) * 256 + c] = ar.store_inv_scaled(v[i]);
    }
}

// ---- row pass: a wave runs its four rows for up to N16_ROWS_GROUP limbs of the same prime (n_here of them, inst_stride
// words apart): the twiddles of the rows -- 15 pairs per row for one step, 15 pairs per thread for the other, more bytes
// than the rows themselves -- are fetched once (LDS and registers), and the next limb's rows are requested before the
// current ones are transformed.  Global traffic is contiguous: the layout of 16 neighbours per thread only touches LDS.
#define N16_ROWS_GROUP 8

template <int S, bool FWD, class A>
__device__ __forceinline__ void rows_body(u64 *g, size_t inst_stride, int n_here, const u64 *tw, const PrimeConst &pc, u64 *lds, ulonglong2 *tw1, int r0) {
    A ar;
    ar.init(pc);
    const int lane = threadIdx.x, rho = lane >> 4, j = lane & 15;
    const u32 base = Ring<S>::ROWS + r0 + rho;
    typename A::T v[16];
    row_table_to_lds(tw1, tw, tw + Ring<S>::N, base, rho, j);
    TwRegs tw2;
    tw2.load(tw, tw + Ring<S>::N, Ring<S>::N, r0 + rho, j);
    const ulonglong2 *tab = tw1 + rho * 16;
    const int at = FWD ? rho * 256 + j : lane;  // forward: value i at j + 16 i of row rho; inverse: at lane + 64 i of the four rows
    constexpr int step = FWD ? 16 : 64;
    u64 nv[16];
#pragma unroll
    for (int i = 0; i < 16; i++) nv[i] = g[at + step * i];
    wave_lds_fence();
#pragma unroll 1
    for (int c = 0; c < n_here; c++) {
        tw2.keep();
        if (FWD) {
#pragma unroll
            for (int i = 0; i < 16; i++) v[i] = ar.load(nv[i]);
        } else {
#pragma unroll
            for (int i = 0; i < 16; i++) lds[rpad(lane + 64 * i)] = nv[i];
        }
        if (c + 1 < n_here) {
            const u64 *gn = g + (size_t)(c + 1) * inst_stride;
#pragma unroll
            for (int i = 0; i < 16; i++) nv[i] = gn[at + step * i];
        }
        u64 *go = g + (size_t)c * inst_stride;
        if (FWD) {
            row_fwd<false>(ar, v, tab, tw2, lds, rho, j);
#pragma unroll
            for (int i = 0; i < 16; i++) lds[rpad(rho * 256 + 16 * j + i)] = ar.store_fwd(v[i]);
            wave_lds_fence();
#pragma unroll
            for (int i = 0; i < 16; i++) go[lane + 64 * i] = lds[rpad(lane + 64 * i)];
            wave_lds_fence();
        } else {
            wave_lds_fence();
#pragma unroll
            for (int i = 0; i < 16; i++) v[i] = ar.center(ar.load(lds[rpad(rho * 256 + 16 * j + i)]));
            wave_lds_fence();
            row_inv(ar, v, tab, tw2, lds, rho, j);
#pragma unroll
            for (int i = 0; i < 16; i++) go[rho * 256 + j + 16 * i] = ar.store_inv(v[i]);
        }
    }
}

template <int S, bool FWD>
__global__ __launch_bounds__(N16_THREADS) void k_ntt16_cols(u64 *data, const u64 *tw_all, const PrimeConst *pcs, LimbMap map) {
    typedef Ring<S> R;
    __shared__ u64 lds[4096];
    const int inst = blockIdx.y;
    const int prime = map.prime[inst % map.n];
    const PrimeConst pc = load_prime(pcs, prime);
    const u64 *tw = tw_all + (size_t)prime * 4 * R::N + (FWD ? 0 : 2 * R::N);
    u64 *g = data + (size_t)inst * R::N + (size_t)blockIdx.x * R::COLS;
    if (pc.kind == PRIME_FP) cols_body<S, FWD, ArithFp>(g, g, tw, pc, lds);
    else if (pc.kind == PRIME_WIDE) cols_body<S, FWD, ArithWide>(g, g, tw, pc, lds);
    else cols_body<S, FWD, ArithInt>(g, g, tw, pc, lds);
}

// Forward column pass that reads every limb from its operand ciphertext and writes the operand array of the
// ciphertext products: row inst = (operand u, polynomial p, limb i) of data <- ops[u].p[p][i], column-transformed.
// l1 limbs per polynomial, limb i under prime i.
template <int S>
__global__ __launch_bounds__(N16_THREADS) void k_ntt16_cols_gather(u64 *data, const MmOperand *ops, int l1, const u64 *tw_all,
                                                                    const PrimeConst *pcs) {
    typedef Ring<S> R;
    __shared__ u64 lds[4096];
    const int inst = blockIdx.y;
    const int u = inst / (2 * l1), y = inst - u * 2 * l1, p = y / l1, prime = y - p * l1;
    const PrimeConst pc = load_prime(pcs, prime);
    const u64 *tw = tw_all + (size_t)prime * 4 * R::N;
    const MmOperand op = ops[u];
    const u64 *gin = op.p + ((size_t)p * op.limb_stride + prime) * R::N + (size_t)blockIdx.x * R::COLS;
    u64 *g = data + (size_t)inst * R::N + (size_t)blockIdx.x * R::COLS;
    if (pc.kind == PRIME_FP) cols_body<S, true, ArithFp>(g, gin, tw, pc, lds);
    else if (pc.kind == PRIME_WIDE) cols_body<S, true, ArithWide>(g, gin, tw, pc, lds);
    else cols_body<S, true, ArithInt>(g, gin, tw, pc, lds);
}

// grid (4 TILES, map.n * n_groups): instance inst = slot + map.n * (N16_ROWS_GROUP * group + c), c < N16_ROWS_GROUP, lies
// under prime map.prime[slot]; n_inst instances in all.
template <int S, bool FWD>
__global__ __launch_bounds__(64, 2) void k_ntt16_rows(u64 *data, const u64 *tw_all, const PrimeConst *pcs, LimbMap map, int n_inst) {
    typedef Ring<S> R;
    __shared__ u64 lds[ROW_LDS];
    __shared__ ulonglong2 tw1[4 * 16];
    const int slot = blockIdx.y % map.n, group = blockIdx.y / map.n;
    const int inst0 = slot + map.n * N16_ROWS_GROUP * group;
    if (inst0 >= n_inst) return;
    const int n_here = min(N16_ROWS_GROUP, (n_inst - inst0 + map.n - 1) / map.n);
    const int prime = map.prime[slot];
    const PrimeConst pc = load_prime(pcs, prime);
    const u64 *tw = tw_all + (size_t)prime * 4 * R::N + (FWD ? 0 : 2 * R::N);
    const int r0 = blockIdx.x * 4;
    u64 *g = data + (size_t)inst0 * R::N + (size_t)r0 * 256;
    const size_t stride = (size_t)map.n * R::N;
    if (pc.kind == PRIME_FP) rows_body<S, FWD, ArithFp>(g, stride, n_here, tw, pc, lds, tw1, r0);
    else if (pc.kind == PRIME_WIDE) rows_body<S, FWD, ArithWide>(g, stride, n_here, tw, pc, lds, tw1, r0);
    else rows_body<S, FWD, ArithInt>(g, stride, n_here, tw, pc, lds, tw1, r0);
}

// Grid of the row pass over n_inst instances whose primes repeat with period `period`.
static dim3 rows_grid(int tiles, int n_inst, int period) {
    const int reps = (n_inst + period - 1) / period;  // instances per prime slot (the last ones may be missing)
    return dim3(4 * tiles, period * ((reps + N16_ROWS_GROUP - 1) / N16_ROWS_GROUP));
}

// Forward transform of n_ops operand ciphertexts (two polynomials of l1 limbs each, limb i under prime i) from where they
// lie into data[n_ops][2][l1][N]: the column pass gathers, the row pass runs in place.  ops: device array.
void launch_ntt16_gather(ensi_ctx *ctx, u64 *data, const MmOperand *ops, int n_ops, int l1, hipStream_t st) {
    LimbMap map;
    map.n = l1;
    for (int e = 0; e < ENSI_MAX_EXT; e++) map.prime[e] = e < l1 ? e : 0;
    const int per = 32768 / (2 * l1);  // operands per launch (grid y below 65536)
    ring_dispatch(ctx->log_n, [&](auto s) {
        constexpr int S = decltype(s)::value, TILES = Ring<S>::TILES;
        for (int done = 0; done < n_ops; done += per) {
            const int cnt = std::min(per, n_ops - done);
            u64 *d = data + (size_t)done * 2 * l1 * ctx->N;
            {
                ScopedTimer t(ctx, "ntt_fwd_cols", st);
                hipLaunchKernelGGL((k_ntt16_cols_gather<S>), dim3(TILES, cnt * 2 * l1), dim3(N16_THREADS), 0, st, d, ops + done, l1, ctx->d_tw, ctx->d_pc);
            }
            {
                ScopedTimer t(ctx, "ntt_fwd_rows", st);
                hipLaunchKernelGGL((k_ntt16_rows<S, true>), rows_grid(TILES, cnt * 2 * l1, map.n), dim3(64), 0, st, d, ctx->d_tw, ctx->d_pc, map, cnt * 2 * l1);
            }
        }
    });
}

void launch_ntt16(ensi_ctx *ctx, u64 *data, int n_inst, const LimbMap &map, bool inverse, hipStream_t st) {
    const int max_rows = (32768 / map.n) * map.n;
    ring_dispatch(ctx->log_n, [&](auto s) {
        constexpr int S = decltype(s)::value, TILES = Ring<S>::TILES;
        for (int done = 0; done < n_inst; done += max_rows) {
            const int cnt = std::min(max_rows, n_inst - done);
            u64 *d = data + (size_t)done * ctx->N;
            const dim3 grid(TILES, cnt), rgrid = rows_grid(TILES, cnt, map.n);
            if (!inverse) {
                {
                    ScopedTimer t(ctx, "ntt_fwd_cols", st);
                    hipLaunchKernelGGL((k_ntt16_cols<S, true>), grid, dim3(N16_THREADS), 0, st, d, ctx->d_tw, ctx->d_pc, map);
                }
                {
                    ScopedTimer t(ctx, "ntt_fwd_rows", st);
                    hipLaunchKernelGGL((k_ntt16_rows<S, true>), rgrid, dim3(64), 0, st, d, ctx->d_tw, ctx->d_pc, map, cnt);
                }
            } else {
                {
                    ScopedTimer t(ctx, "ntt_inv_rows", st);
                    hipLaunchKernelGGL((k_ntt16_rows<S, false>), rgrid, dim3(64), 0, st, d, ctx->d_tw, ctx->d_pc, map, cnt);
                }
                {
                    ScopedTimer t(ctx, "ntt_inv_cols", st);
                    hipLaunchKernelGGL((k_ntt16_cols<S, false>), grid, dim3(N16_THREADS), 0, st, d, ctx->d_tw, ctx->d_pc, map);
                }
            }
        }
    });
}
