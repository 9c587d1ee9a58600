// Alg. 1 (PCMM) as a dense integer contraction on the matrix cores.
//
// y_i = sum_v W'[v][i] * x_v over limb words, W' in {-1,0,+1}.  The paper's point is
// that these products need no ciphertext multiplication; on this chip the cheapest
// way to form the signed sums is still the int8 matrix pipe: every 64-bit limb word
// is split into byte planes, each plane is contracted against the ternary weights
// with V_MFMA_I32_32X32X32_I8 (exact 32-bit integer sums), and the planes are
// recombined with shifts and reduced mod q once per output word.  The result is
// bit-identical to the sequence of modular additions and subtractions.
//
// The chip is bound by power in this kernel, and what an instruction draws hangs on its data: signed bytes times signed
// weights keep the sign extensions of products and sums flipping.  Where the primes allow it the digits and the weights
// are therefore made non-negative (AM_POS7: primes below 2^36 and 2^50): planes of 7 bits below a top plane of 8, weights
// w + 1 in {0, 1, 2}, and the sum of all operands, one per word (`word sums`), taken off again when the planes are
// recombined.  An LDS-fed loop of the instruction alone: 19.8 ns each on signed bytes and weights, 19.3 with the weights shifted,
// 17.0 with both (the same digits and signed weights: 19.8).  A step of the kernel: 0.312 us before, 0.276 with them.
// Primes between (37 to 40 bits: five planes of 8 bits, seven of 7), primes above 2^50, products of up to AM_POS7_MIN operands,
// where an item is mostly its recombination, and products of few outputs or few words, which the sum of the operands costs more than
// it saves, use 8-bit planes and signed weights (AM_FP8, AM_INT8).
//
// The matrix pipe is signed: an 8-bit digit u is fed as u-128 (u xor 0x80), and 128 times the sum of the weights of output i
// (`bias`) is added back to its plane when the planes are recombined.
//
// Operand v is the ciphertext at xbase + v*xstride words (the unpack phase writes its
// rotations straight into that array).
//
// Products of few operands or few outputs run in one kernel, k_accumulate_direct, which keeps its digits in LDS; the others in two.
// k_byte_planes runs once per operand array: it splits every 32 x 32 tile
// (32 operands x 32 consecutive words) into its byte planes, already in the register
// layout of the matrix instruction's first operand (lane = 32*(operand/16) + row, 16
// operand bytes per lane; plane_row says which word a row is), so that the tile of one plane is 1 KiB that a single
// asynchronous global->LDS copy drops in place.  Tiles are stored [word tile][step]
// [plane]: a work item of the contraction streams one contiguous run.  The split is done
// once instead of once per output tile (10 to 27 times at the benchmark shapes), which
// takes the byte shuffling, the plane stores and a second LDS buffer out of the
// contraction's inner loop.  The plane array of a whole operand array can exceed the
// memory left, so the host works through the coefficients in slices (a slice holds a
// range of 32-coefficient tiles of every limb of both polynomials).  The split can apply
// the scalar-multiply + rescale step between two layers on the fly (k_byte_planes_rescale):
// the rescaled operands then never exist as 64-bit words in memory.
//
// k_accumulate_mfma.  A work item is 256 outputs x 32 consecutive words; inside it each
// of the 4 waves owns 64 outputs (two 32x32 blocks) for all byte planes and walks the
// operands in steps of 32.  Per step:
//   * the step's plane tiles and the wave's two weight fragments arrive in LDS by
//     asynchronous global->LDS copies issued AM_RING steps earlier (rings of AM_RING
//     slots; no registers are held while they are in flight);
//   * the fragments of step k+1 are read from LDS while the matrix instructions of
//     step k run from registers;
//   * one barrier.
// The words are the first operand of the matrix instruction and the weights the second: under this load the chip is bound by
// power, and a register-only loop on random bytes and ternary weights takes 41.1 cycles (of 2.4 GHz) per instruction this way
// round against 46.3 the other.
// An item costs 5.2 us besides its steps, in a fit over 8 to 128 steps; without its stores 2.8, without its recombination 4.5,
// without both 1.4.  The stores are bound by what the CUs of an XCD, which run in step, can write at once; spread over
// the next item's steps (from registers) they cost more, 6 us, because a copy is not seen to have landed before the stores
// issued ahead of it are done.
// The step loop holds no vector-ALU instruction besides the matrix instructions: the running source addresses of the
// copies are wave-uniform and live in scalar registers (a lane adds 16 * lane through the instruction's offset
// operand).  Vector instructions issued between matrix instructions slow the matrix pipe down measurably -- four 64-bit
// address updates per step cost 5 % of the kernel, an in-loop unpacking of 2-bit weights (22 instructions) 10 %.
// The grid is persistent: one workgroup per CU, 32 per XCD.  Items that share their
// 32 words (different output tiles) are consecutive in one XCD's list and the
// workers of that XCD take the list round-robin, so they read the same plane tiles
// at nearly the same time and all but the first read are served by that XCD's L2.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "ntt16_core.h"

#include <ensi_dma.h>

typedef int v4i __attribute__((vector_size(16)));
typedef int v16i __attribute__((vector_size(64)));

#define AM_THREADS 256
#define AM_TILE_M 256
#define AM_TILE_N 32
#define AM_TILE_K 32
#define AM_DEPTH 7
#define AM_RING (AM_DEPTH + 1)  // power of two; the step loop is unrolled by it so every LDS offset is a constant
#define AM_BSLOT 8192           // plane tiles of one step (1 KiB each, PLANES of 8 used)
#define AM_ASLOT 2048           // one wave's two weight fragments of one step

// The word sums of an item are copied to one of two slots by all four waves while the item before it is multiplied: the slot's last
// readers have finished only if an item is more than one group of steps (AM_RING), which more than AM_POS7_MIN operands fill.
static_assert(AM_POS7_MIN >= AM_RING * AM_TILE_K, "an item with word sums must be more than one group of steps");

#define AM_STORES 16            // stores of one item by one wave: 64 outputs x 32 words, 1 KiB each
#define AM_OROW 144             // 16 words of an output, padded

// Byte b of four dwords gathered into one dword (4x4 byte transpose, two stages).
__device__ __forceinline__ void transpose4(u32 a0, u32 a1, u32 a2, u32 a3, u32 *p) {
    u32 t0 = __builtin_amdgcn_perm(a1, a0, 0x05010400u);
    u32 t1 = __builtin_amdgcn_perm(a1, a0, 0x07030602u);
    u32 t2 = __builtin_amdgcn_perm(a3, a2, 0x05010400u);
    u32 t3 = __builtin_amdgcn_perm(a3, a2, 0x07030602u);
    p[0] = __builtin_amdgcn_perm(t2, t0, 0x05040100u);
    p[1] = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
    p[2] = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
    p[3] = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
}

// signed 64-bit T (|T| < 2^63, |T|/q < 2^31) to its canonical residue mod q
__device__ __forceinline__ u64 reduce_signed(int64_t t, u64 q, double q_inv) {
    const int k = (int)rint((double)t * q_inv);
    int64_t r = t - (int64_t)k * (int64_t)q;
    if (r < 0) r += (int64_t)q;
    if (r < 0) r += (int64_t)q;
    if (r >= (int64_t)q) r -= (int64_t)q;
    return (u64)r;
}

// The same recombination for primes below 2^50, in double precision on exact integers (no 64-bit integer
// multiplies, which take many quarter-rate instructions on this chip).  S_p: the plane sums from the matrix
// pipe; the true plane sums are T_p = S_p + b with b = 128 * (column sum of the weights), and the result is
// sum_p T_p 2^(8p) mod q = (sum_p S_p 2^(8p) + B) mod q with B = b * sum_p 2^(8p) mod q, which the host supplies
// per output and limb as a double in [0, q).  |S_p| <= 2^22 for up to 32768 operands, so planes are first paired
// in 32-bit integers (S_p + 2^8 S_(p+1) < 2^31) and the pairs combined into lo + 2^32 hi with |lo| < 2^48 and
// |hi| < 2^38.1 -- every product by a power of two and every sum below 2^53 is exact in a double.  One reduction:
// k = rint((lo + B + 2^32 hi) / q), whose argument is off by its three roundings, 3 2^-53 |k| at most: below 2^-9 for the smallest
// primes (2^13 < q, |k| < 2^42), 2^-26 at 41 bits and 32768 operands.  Then 2^32 hi - k q, an integer below 2^52 in magnitude
// that the fused multiply-add returns exactly (as a multiple of 2^-32: hi - k (q 2^-32)), plus lo + B: a representative within
// (1/2 + 2^-9) q of zero -- below q in magnitude is all that is needed -- shifted into [0, q).
// AM_POS7: the same with 2^7 for 2^8.  Only the top plane has an offset; B is that offset 128 2^(7 (PLANES - 1)) (sum of the
// weights) mod q less the word sum mod q, |B| < q.  |S_p| <= 2^23, so a pair stays below 2^31, lo below 2^45, hi below 2^38.
struct AmModulus {
    double q, q_inv, q_lo, q_inv_hi;  // q and 1/q; q / P4 and P4 / q
};
template <bool POS7>
struct AmDigits {
    static constexpr int BITS = POS7 ? 7 : 8;
    static constexpr double P2 = 1 << 2 * BITS, P4 = (double)((int64_t)1 << 4 * BITS);
};
template <int PLANES, bool POS7>
__device__ __forceinline__ u64 recombine_fp(const int (&S)[PLANES], double B, const AmModulus &m) {
    constexpr int DB = AmDigits<POS7>::BITS;
    constexpr double P2 = AmDigits<POS7>::P2, P4 = AmDigits<POS7>::P4;
    const int c01 = S[0] + (S[1] << DB), c23 = S[2] + (S[3] << DB);
    const double lb = fma((double)c23, P2, (double)c01) + B;
    double hi;
    if (PLANES == 7) {
        const int c45 = S[4] + (S[5] << DB);
        hi = fma((double)S[6], P2, (double)c45);
    } else {
        hi = (double)S[4];
    }
    const double k = rint(fma(lb, m.q_inv, hi * m.q_inv_hi));
    double u = fma(fma(-k, m.q_lo, hi), P4, lb);
    u = u < 0.0 ? u + m.q : u;
    // an integer in [0, 2^52) plus 2^52 has that integer as its mantissa
    return (u64)__double_as_longlong(u + 4503599627370496.0) & 0xFFFFFFFFFFFFFull;
}

// ---------------------------------------------------------------- byte planes of the operands
// Digits of a word, one per byte: planes 0 .. 3 in d[0], the rest in d[1].
template <int PLANES, bool POS7>
__device__ __forceinline__ void digits(u64 w, u32 *d) {
    if (!POS7) {
        d[0] = (u32)w;
        d[1] = (u32)(w >> 32);
        return;
    }
    // 28 bits as two halves of 14 sixteen bits apart, each then as two digits of 7 eight bits apart
    auto bfi = [](u32 m, u32 a, u32 b) { return (a & m) | (b & ~m); };
    const u32 lo = bfi(0x3fffu, (u32)w, (u32)w << 2);
    d[0] = bfi(0x007f007fu, lo, lo << 1) & 0x7f7f7f7fu;
    const u32 h = (u32)(w >> 28);
    if (PLANES == 5) {
        d[1] = h;  // the top digit alone
    } else {
        const u32 hi = bfi(0x3fffu, h, h << 2);  // bits 16 up: the top digit
        d[1] = bfi(0x7f00u, hi << 1, hi) & 0x00ff7f7fu;
    }
}

// Slice-local word tile: nt_local = pl * cw + ctile, pl = poly * l1 + limb, ctile = coefficient tile - c0.
// Thread (k4 = tid / 32, ln = tid % 32) handles operands 4*k4 .. 4*k4+3 of a step, word ln: its four
// words give one dword (4 operand bytes) of every plane.  A plane tile is staged in LDS and written out as
// whole 16-byte lane entries.  Digits of 8 bits are stored as u - 128 (u xor 0x80), those of 7 as they are; operands beyond n_v
// are zero words.
// Row of the plane tile that holds word ln: accumulator register r of a lane is row 8*(r/4) + 4*(lane/32) + r%4 and holds
// word 16*(r/8) + 8*(lane/32) + r%8, so that the two lanes of an output hold 16 consecutive words in eight registers.
__device__ __forceinline__ int plane_row(int ln) { return ((ln >> 4) * 2 + ((ln >> 2) & 1)) * 8 + ((ln >> 3) & 1) * 4 + (ln & 3); }

struct AmFp {  // fp64 arithmetic on exact integers modulo a prime below 2^50 (as in the rescale kernel)
    double q, qinv;
    __device__ __forceinline__ double mid(double x) const { return fma(-rint(x * qinv), q, x); }
    __device__ __forceinline__ double mulmod(double x, double w, double wq) const {
        const double h = x * w;
        const double l = fma(x, w, -h);
        const double t = rint(x * wq);
        return fma(-t, q, h) + l;
    }
};

// red (POS7): the sum of the thread's operands, complete for the block after the first barrier.
template <int PLANES, bool POS7, int STEPS>
__device__ __forceinline__ void planes_out(const u64 (&w)[STEPS][4], u32 (*stage)[PLANES * 256], int dst, v4i *out, int tid, u64 *red) {
    if (POS7) {
        u64 t = 0;
#pragma unroll
        for (int s8 = 0; s8 < STEPS; s8++) t += (w[s8][0] + w[s8][1]) + (w[s8][2] + w[s8][3]);
        red[tid] = t;
    }
#pragma unroll
    for (int s8 = 0; s8 < STEPS; s8++) {
        u32 pl[8], d[4][2];
#pragma unroll
        for (int j = 0; j < 4; j++) digits<PLANES, POS7>(w[s8][j], d[j]);
        transpose4(d[0][0], d[1][0], d[2][0], d[3][0], pl);
        transpose4(d[0][1], d[1][1], d[2][1], d[3][1], pl + 4);
        u32 *st = stage[s8 & 1];
#pragma unroll
        for (int p = 0; p < PLANES; p++) st[p * 256 + dst] = POS7 && p < PLANES - 1 ? pl[p] : pl[p] ^ 0x80808080u;
        __syncthreads();  // (the other staging buffer was read before the previous barrier)
        const v4i *sv = (const v4i *)st;
        for (int e = tid; e < PLANES * 64; e += AM_THREADS) out[(size_t)s8 * PLANES * 64 + e] = sv[e];
    }
}

// Sum of a block's operands at each of its 32 words (red: of each thread's operands) -> part[0 .. 32).  Exact: the operands of a
// product sum to less than 2^63.
__device__ __forceinline__ void word_sums_out(const u64 *red, u64 *part, int tid) {
    if (tid < AM_TILE_N) {
        u64 t = red[tid];
#pragma unroll
        for (int k = 1; k < AM_THREADS / AM_TILE_N; k++) t += red[k * AM_TILE_N + tid];
        part[tid] = t;
    }
}
// part: [word tile][parts][32] -> tsum: [word tile][32] residues modulo the tile's prime, as doubles.  grid (n_tiles * 32 / AM_THREADS)
__global__ __launch_bounds__(AM_THREADS) void k_word_sums(const u64 *part, int parts, int n_words, int cw, int l1, const PrimeConst *pc, double *tsum) {
    const int i = blockIdx.x * AM_THREADS + threadIdx.x, tile = i / AM_TILE_N;
    if (i >= n_words) return;
    const u64 *p = part + (size_t)tile * parts * AM_TILE_N + i % AM_TILE_N;
    u64 t = 0;
    for (int k = 0; k < parts; k++) t += p[k * AM_TILE_N];
    const u64 q = pc[tile / cw % l1].q;
    tsum[i] = (double)reduce_signed((int64_t)t, q, 1.0 / (double)q);
}

// grid (cw, nk / 8, 2 * l1); each block converts 8 steps of one word tile.  POS7: part receives the block's word sums.
template <int PLANES, bool POS7>
__global__ __launch_bounds__(AM_THREADS) void k_byte_planes(const u64 *xbase, u32 xstride, int n_v, int nk, int N, int l1, int limb_stride_in,
                                                            int c0, int cw, char *xp, u64 *part) {
    __shared__ u32 stage[2][PLANES * 256];
    __shared__ u64 red[POS7 ? AM_THREADS : 1];
    const int tid = threadIdx.x, k4 = tid >> 5, ln = tid & 31;
    const int pl = blockIdx.z, poly = pl / l1, limb = pl - poly * l1;
    const u64 *xw = xbase + ((size_t)poly * limb_stride_in + limb) * N + (size_t)(c0 + blockIdx.x) * AM_TILE_N + ln;
    // destination dword of this thread inside a plane tile: lane (k4/4)*32 + ln, dword k4 % 4
    const int dst = ((k4 >> 2) * 32 + plane_row(ln)) * 4 + (k4 & 3);
    v4i *out = (v4i *)(xp + (((size_t)pl * cw + blockIdx.x) * nk + (size_t)blockIdx.y * 8) * PLANES * 1024);
    // all 32 words of the block's 8 steps are requested before the first is used
    u64 w[8][4];
#pragma unroll
    for (int s8 = 0; s8 < 8; s8++)
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int v = (blockIdx.y * 8 + s8) * AM_TILE_K + 4 * k4 + j;
            w[s8][j] = v < n_v ? xw[(size_t)v * xstride] : 0;
        }
    planes_out<PLANES, POS7, 8>(w, stage, dst, out, tid, red);
    if (POS7) word_sums_out(red, part + (((size_t)pl * cw + blockIdx.x) * gridDim.y + blockIdx.y) * AM_TILE_N, tid);
}

// The same with the scalar-multiply + rescale step applied on the way: the operands are read at l1 + 1
// limbs, c <- c * k, limb l1 dropped with rounding to nearest (c_i <- (c_i k - [c_l k]) q_l^-1 mod q_i with
// the centred representative of limb l1), and the planes of the l1 remaining limbs written.  fc: [5][l1+1]
// doubles: k mod q_i, that / q_i, q_l^-1 mod q_i, that / q_i, 1 / q_i.  grid (cw, nk / 4, 2): a block keeps
// the centred last-limb residues of its 32 coefficients x 128 operands in registers and walks the limbs
// (4 steps per block keep the register count low enough for four blocks per CU, or for three where all digits are of 8 bits: two
// registers more than four blocks have, 512 operands at 15 limbs 2.88 against 3.0 ms with those two spilled).
#define AM_RS_STEPS 4
template <int PLANES, bool POS7>
__global__ __launch_bounds__(AM_THREADS, POS7 ? 4 : 3) void k_byte_planes_rescale(const u64 *xbase, u32 xstride, int n_v, int nk, int N, int l1,
                                                                    int limb_stride_in, int c0, int cw, char *xp, const PrimeConst *pc,
                                                                    const double *fc, u64 *part) {
    __shared__ u32 stage[2][PLANES * 256];
    __shared__ u64 red[POS7 ? AM_THREADS : 1];
    const int tid = threadIdx.x, k4 = tid >> 5, ln = tid & 31;
    const int poly = blockIdx.z, lin = l1 + 1;
    const u64 *xw = xbase + (size_t)poly * limb_stride_in * N + (size_t)(c0 + blockIdx.x) * AM_TILE_N + ln;
    const int dst = ((k4 >> 2) * 32 + plane_row(ln)) * 4 + (k4 & 3);
    u64 w[AM_RS_STEPS][4];
    double xl[AM_RS_STEPS][4];
    // operand rows of this thread: row[s8] + j * xstride for j < n_live[s8] (a multiple of four operands except in
    // the last step of a ragged operand count; dead operands re-read row j = 0 and are zeroed before the split)
    const u64 *row[AM_RS_STEPS];
    int n_live[AM_RS_STEPS];
#pragma unroll
    for (int s8 = 0; s8 < AM_RS_STEPS; s8++) {
        const int v0 = (blockIdx.y * AM_RS_STEPS + s8) * AM_TILE_K + 4 * k4;
        n_live[s8] = min(max(n_v - v0, 0), 4);
        row[s8] = xw + (size_t)(n_live[s8] ? v0 : 0) * xstride;
    }
    {
        const AmFp ml = {(double)pc[l1].q, fc[4 * lin + l1]};
        const double kl = fc[l1], kl_q = fc[lin + l1];
#pragma unroll
        for (int s8 = 0; s8 < AM_RS_STEPS; s8++)
#pragma unroll
            for (int j = 0; j < 4; j++) w[s8][j] = row[s8][(size_t)(j < n_live[s8] ? j : 0) * xstride + (size_t)l1 * N];
#pragma unroll
        for (int s8 = 0; s8 < AM_RS_STEPS; s8++)
#pragma unroll
            for (int j = 0; j < 4; j++) xl[s8][j] = ml.mid(ml.mulmod((double)w[s8][j], kl, kl_q));
    }
    for (int limb = 0; limb < l1; limb++) {
        const AmFp m = {(double)pc[limb].q, fc[4 * lin + limb]};
        const double k = fc[limb], k_q = fc[lin + limb], qi = fc[2 * lin + limb], qi_q = fc[3 * lin + limb];
#pragma unroll
        for (int s8 = 0; s8 < AM_RS_STEPS; s8++)
#pragma unroll
            for (int j = 0; j < 4; j++) w[s8][j] = row[s8][(size_t)(j < n_live[s8] ? j : 0) * xstride + (size_t)limb * N];
#pragma unroll
        for (int s8 = 0; s8 < AM_RS_STEPS; s8++)
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const double t = m.mulmod((double)w[s8][j], k, k_q) - m.mid(xl[s8][j]);
                double r = m.mid(m.mulmod(m.mid(t), qi, qi_q));
                r = r < 0.0 ? r + m.q : r;
                w[s8][j] = j < n_live[s8] ? (u64)r : 0;
            }
        v4i *out = (v4i *)(xp + ((((size_t)poly * l1 + limb) * cw + blockIdx.x) * nk + (size_t)blockIdx.y * AM_RS_STEPS) * PLANES * 1024);
        __syncthreads();  // the staging buffers of the previous limb have been written out, its word sums read
        planes_out<PLANES, POS7, AM_RS_STEPS>(w, stage, dst, out, tid, red);
        if (POS7) word_sums_out(red, part + ((((size_t)poly * l1 + limb) * cw + blockIdx.x) * gridDim.y + blockIdx.y) * AM_TILE_N, tid);
    }
}

// primes of the active limbs and their reciprocals, passed by value so that the recombination reads them with
// scalar loads (a vector load there would make the compiler wait for every copy in flight)
struct AmPrimes {
    u64 q[ENSI_MAX_EXT];
    double q_inv[ENSI_MAX_EXT];
};

template <int PLANES>
struct AmLayout {
    static constexpr int bring_off = 0;                                  // [AM_RING][AM_BSLOT]
    static constexpr int aring_off = bring_off + AM_RING * AM_BSLOT;     // [4 waves][AM_RING][AM_ASLOT]
    static constexpr int bias_off = aring_off + 4 * AM_RING * AM_ASLOT;  // [2][256] offset terms of an item's outputs (int32 or double)
    static constexpr int tsum_off = bias_off + 2 * AM_TILE_M * 8;        // [2][32] word sums of an item (doubles; AM_POS7)
    static constexpr int out_off = tsum_off + 2 * AM_TILE_N * 8;             // [4 waves][32 outputs][AM_OROW] results on their way out
    static constexpr int total = out_off + 4 * 32 * AM_OROW;
};

// xp: plane tiles of the slice, [word tile][nk][PLANES][1024]; the slice covers coefficient tiles c0 .. c0+cw-1
// of all 2*l1 limb rows (n_tiles_n = 2*l1*cw word tiles); nk = n_kpad / 32, a multiple of AM_RING.
// MODE AM_POS7, AM_FP8: every active prime is below 2^50, so the planes are recombined in double precision (recombine_fp) and
// bias points to doubles [l1][n_tiles_m * 256], the offset term of every output reduced modulo each limb's prime; AM_INT8:
// the planes are recombined in 64-bit integers and bias points to int32 [n_tiles_m * 256], 128 * column sum of the weights.
// tsum (AM_POS7): the word sums, [word tile][32].
template <int PLANES, int MODE>
__global__ __launch_bounds__(AM_THREADS) void k_accumulate_mfma(const char *xp, int c0, int cw, int n_kpad, const v4i *wfrag, const void *bias,
                                                                const double *tsum, int m, AmPrimes pr, int N, int l1, u64 *out, int limb_stride_out,
                                                                int n_tiles_n, int n_tiles_m, int workers_per_xcd, int m_group) {
    HIP_DYNAMIC_SHARED(char, smem)
    typedef AmLayout<PLANES> LY;
    constexpr bool FP_EPI = MODE != AM_INT8, POS7 = MODE == AM_POS7;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5, nl = lane & 31;
    const int nk = n_kpad / AM_TILE_K;
    const u32 smem0 = lds_addr(smem);
    // the wave copies plane tiles pb0 and pb1 of every step (the last plane twice where 2*wave+1 runs past it)
    const int pb0 = 2 * wv < PLANES ? 2 * wv : PLANES - 1, pb1 = 2 * wv + 1 < PLANES ? 2 * wv + 1 : PLANES - 1;
    // wave-uniform LDS byte addresses of this wave's copy targets (slot 0)
    const u32 b_lds0 = (u32)__builtin_amdgcn_readfirstlane((int)(smem0 + LY::bring_off + pb0 * 1024));
    const u32 b_lds1 = (u32)__builtin_amdgcn_readfirstlane((int)(smem0 + LY::bring_off + pb1 * 1024));
    const u32 a_lds = (u32)__builtin_amdgcn_readfirstlane((int)(smem0 + LY::aring_off + wv * AM_RING * AM_ASLOT));
    const char *a_rd = smem + LY::aring_off + wv * AM_RING * AM_ASLOT + lane * 16;
    const char *b_rd = smem + LY::bring_off + lane * 16;
    char *o_lds = smem + LY::out_off + wv * 32 * AM_OROW;
    const size_t ct_words_out = (size_t)2 * limb_stride_out * N;
    const int xcd = blockIdx.x & 7, worker = blockIdx.x >> 3;
    const int n_nt = (n_tiles_n + 7) / 8;  // word tiles of this XCD
    const int per_group = n_nt * m_group, last_group = (n_tiles_m - 1) / m_group, last_size = n_tiles_m - last_group * m_group;

    // Items are ordered: group of m_group output tiles, word tile, output tile inside the group; the workers of an
    // XCD therefore share both plane tiles and weight fragments through its L2.  A workgroup steps through its items with
    // (group, place in the group); dividing by the group's size takes one multiplication by a rounded-up reciprocal, exact
    // for places below 2^29 / 8 (an item's address arithmetic sits between its matrix instructions and the next item's).
    const u32 recip_full = 0xffffffffu / (u32)m_group + 1, recip_last = 0xffffffffu / (u32)last_size + 1;  // (unused for a size of one)
    struct Item {
        int mg, j;            // group of output tiles, place in it
        int m_tile, nt_local;  // output tile, word tile of the slice
    };
    // item at or after place (mg, j) that is not one of the padding slots of the last group of 8 word tiles
    auto settle = [&](Item &t) {
        for (;; t.j += workers_per_xcd) {
            while (t.mg < last_group && t.j >= per_group) {
                t.j -= per_group;
                t.mg++;
            }
            const int size = t.mg < last_group ? m_group : last_size;
            if (t.mg >= last_group && t.j >= n_nt * size) return false;
            const int col = size == 1 ? t.j : (int)__umulhi((u32)t.j, t.mg < last_group ? recip_full : recip_last);
            t.m_tile = t.mg * m_group + t.j - col * size;
            t.nt_local = col * 8 + xcd;
            if (t.nt_local < n_tiles_n) return true;
        }
    };

    // The copies of all items of this workgroup form one stream of steps: the ring never drains between items.
    // pb/pa are the running per-lane source pointers of the stream.
    // pb/pa are wave-uniform (scalar registers, advanced by the scalar unit); a lane adds its own 16 * lane bytes.
    const char *pb[2], *pa;
    const u32 lane_off = (u32)lane * 16;
    auto seek = [&](const Item &t) {
        const char *pbase = xp + (size_t)t.nt_local * nk * PLANES * 1024;
        pb[0] = pbase + pb0 * 1024;
        pb[1] = pbase + pb1 * 1024;
        pa = (const char *)(wfrag + ((size_t)t.m_tile * nk * 4 + wv) * 128);
    };
    // one of the wave's two plane tiles of the stream's next step -> ring slot
    auto issue_b = [&](int slot, int c) {
        dma_load16_s(pb[c], lane_off, (c ? b_lds1 : b_lds0) + (u32)slot * AM_BSLOT);
        pb[c] += PLANES * 1024;
    };
    // one of the wave's two weight fragments of the stream's next step -> ring slot
    auto issue_a = [&](int slot, int c) {
        dma_load16_s(pa + c * 1024, lane_off, a_lds + (u32)slot * AM_ASLOT + c * 1024);
        if (c == 1) pa += 8192;
    };

    // offset terms of an item's 256 outputs -> one of two LDS buffers (64 per wave); issued one item ahead
    constexpr int BIAS_BYTES = FP_EPI ? 8 : 4;
    const u32 bias_lds = (u32)__builtin_amdgcn_readfirstlane((int)(smem0 + LY::bias_off + wv * 64 * BIAS_BYTES));
    const u32 recip_cw = 0xffffffffu / (u32)cw + 1;  // limb row of a word tile: exact for 2^16 tiles and cw up to 2^15
    auto limb_row = [&](const Item &t) { return cw == 1 ? t.nt_local : (int)__umulhi((u32)t.nt_local, recip_cw); };
    const u32 tsum_lds = (u32)__builtin_amdgcn_readfirstlane((int)(smem0 + LY::tsum_off));
    auto issue_bias = [&](const Item &t, int buf) {
        // (the word sums: every wave copies the same 256 bytes to the same place, and waits for its own copy only.  An item of more
        // than one group of steps begins long after every wave has read those of the item before the last.)
        if (POS7) dma_load4((const char *)(tsum + (size_t)t.nt_local * AM_TILE_N) + lane * 4, tsum_lds + (u32)buf * (AM_TILE_N * 8));
        if (FP_EPI) {
            // the wave's 64 doubles of the item's limb, as two copies of 4 bytes per lane (256 contiguous bytes each)
            const int pl = limb_row(t), limb = pl < l1 ? pl : pl - l1;
            const char *src = (const char *)((const double *)bias + (size_t)limb * n_tiles_m * AM_TILE_M + t.m_tile * AM_TILE_M + wv * 64) + lane * 4;
            dma_load4(src, bias_lds + (u32)buf * (AM_TILE_M * 8));
            dma_load4(src + 256, bias_lds + (u32)buf * (AM_TILE_M * 8) + 256);
        } else {
            dma_load4((const int32_t *)bias + t.m_tile * AM_TILE_M + wv * 64 + lane, bias_lds + (u32)buf * (AM_TILE_M * 4));
        }
    };

    Item item = {0, worker, 0, 0};
    if (!settle(item)) return;
    issue_bias(item, 0);
    // Copies are issued in one fixed order, "iteration j issues B(j+8) then A(j+8) into slot j % 8" (j counts the
    // steps of the stream), from j = -8 on, so that waiting until at most 24 copies are outstanding always means:
    // everything of iteration j-6 has landed.
    seek(item);
#pragma unroll
    for (int t = 0; t < AM_RING; t++) {  // iterations -8 .. -1: steps 0..7 of the first item
        issue_b(t, 0);
        issue_b(t, 1);
        issue_a(t, 0);
        issue_a(t, 1);
    }
    wait_vmcnt<4 * (AM_DEPTH - 1)>();  // steps 0 and 1 have landed
    __syncthreads();
    // Fragments live in two register sets used alternately: step ks multiplies from set ks & 1 while the
    // fragments of step ks+1 are read into the other set.  (With one set, the LDS read that refills a
    // fragment's registers has to wait for the matrix instructions still reading them, and every later
    // instruction of the wave queues behind it.)  nk is even, so every item starts on set 0.
    v4i bf[2][PLANES], af[2][2];
#pragma unroll
    for (int p = 0; p < PLANES; p++) bf[0][p] = *(const v4i *)(b_rd + p * 1024);
    af[0][0] = *(const v4i *)a_rd;
    af[0][1] = *(const v4i *)(a_rd + 1024);
    __syncthreads();  // slot 0 has been read by every wave before step 0 refills it

    bool stores_pending = false;  // the previous item's AM_STORES stores of this wave may still be on their way
    bool more = true;
    for (int it = 0; more; it++) {
        Item next = {item.mg, item.j + workers_per_xcd, 0, 0};
        more = settle(next);
        const int pl = limb_row(item), poly = pl >= l1, limb = poly ? pl - l1 : pl;
        const size_t off_out = ((size_t)poly * limb_stride_out + limb) * N + (size_t)(c0 + item.nt_local - pl * cw) * AM_TILE_N;
        const int i0 = item.m_tile * AM_TILE_M + wv * 64;
        // offset terms of this item's outputs: copied one item ahead into two buffers used alternately (the
        // other one may still be read by a wave that has not finished the previous item's recombination)
        const char *bl = smem + LY::bias_off + (it & 1) * AM_TILE_M * BIAS_BYTES;
        const double *tl = (const double *)(smem + LY::tsum_off) + (it & 1) * AM_TILE_N;

        v16i acc[PLANES][2];
        // Step ks multiplies from registers filled during step ks-1; meanwhile it reads the fragments of step
        // ks+1 from slot (ks+1) % RING and issues the copies of the stream's step ks+8 into slot ks % RING (read
        // during step ks-1, before the barrier that ended it).  During the last 8 steps of an item the stream
        // has moved on to the first 8 steps of the next item (after the last item: of the same item again,
        // which nobody reads).  Scheduling fences keep the LDS reads and the copies spread between the matrix
        // instructions.
        auto steps = [&](int ks0, auto first_group) {
            constexpr bool FIRST = decltype(first_group)::value;
            if (ks0 + AM_RING == nk) {
                seek(more ? next : item);
                if (more) issue_bias(next, (it + 1) & 1);
            }
#pragma unroll
            for (int s = 0; s < AM_RING; s++) {
                const int cur = s & 1, nxt = cur ^ 1;
                const char *brn = b_rd + ((s + 1) % AM_RING) * AM_BSLOT;
                const char *arn = a_rd + ((s + 1) % AM_RING) * AM_ASLOT;
                af[nxt][0] = *(const v4i *)arn;
                af[nxt][1] = *(const v4i *)(arn + 1024);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int p = 0; p < PLANES; p++) {
                    bf[nxt][p] = *(const v4i *)(brn + p * 1024);
                    __builtin_amdgcn_sched_barrier(0);
                    // (the first step adds to the constant zero: clearing 32 registers a plane by hand is not hidden)
                    const v16i zero = {};
                    acc[p][0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(bf[cur][p], af[cur][0], FIRST && s == 0 ? zero : acc[p][0], 0, 0, 0);
                    acc[p][1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(bf[cur][p], af[cur][1], FIRST && s == 0 ? zero : acc[p][1], 0, 0, 0);
                    if (p == 0) issue_b(s, 0);
                    if (p == 1) issue_b(s, 1);
                    if (p == 2) issue_a(s, 0);
                    if (p == 3) issue_a(s, 1);
                    __builtin_amdgcn_sched_barrier(0);
                }
                // keep this step's fragments alive up to here, so that the register allocator cannot hand
                // their registers to the next step's fragments while matrix instructions still read them
#pragma unroll
                for (int p = 0; p < PLANES; p++) asm volatile("" ::"v"(bf[cur][p]));
                asm volatile("" ::"v"(af[cur][0]), "v"(af[cur][1]));
                // Step ks+2 has landed once at most six iterations' copies are outstanding.  The counter goes down in the order
                // of issue, and the AM_STORES stores of the previous item's recombination lie between its last copies and
                // this item's first: for six steps they may be outstanding as well, so that no step waits for memory to
                // take them (waiting at the first step cost 3 % of a 1536 x 4096 product on 2^21 words, 149 -> 145 ms for two).
                if (FIRST && s < AM_DEPTH - 1 && stores_pending) wait_vmcnt<4 * (AM_DEPTH - 1) + AM_STORES>();
                else wait_vmcnt<4 * (AM_DEPTH - 1)>();
                __syncthreads();
            }
        };
        steps(0, std::true_type());
        for (int ks0 = AM_RING; ks0 < nk; ks0 += AM_RING) steps(ks0, std::false_type());
        // here bf[0]/af[0] already hold step 0 of the next item

        // Recombine planes, add the offset term of the output, take off the word sum, reduce mod q, store.
        // Accumulator register r of a lane holds output lane%32 of the block, word 16*(r/8) + 8*(lane/32) + r%8 (plane_row).
        // 32 outputs x 16 words at a time pass through LDS so that a store writes whole lines: outputs lie a power of two
        // apart, and stores of 16 bytes to each of 32 of them at once all went to one L2 channel.
        // While one piece is on its way through LDS the next one is recombined.
        const u64 q = pr.q[limb];
        const double q_inv = pr.q_inv[limb], qd = (double)q;
        const AmModulus md = {qd, q_inv, qd / AmDigits<POS7>::P4, q_inv * AmDigits<POS7>::P4};
        u64 ones = 0;
#pragma unroll
        for (int p = 0; p < PLANES; p++) ones |= (u64)1 << (8 * p);
        const bool whole = i0 + 64 <= m;  // all 64 outputs of this wave exist (wave-uniform): stores need no bounds check
        u64 res[4][2];
        auto piece = [&](int mb, int h) {
            const double b_fp = FP_EPI ? ((const double *)bl)[wv * 64 + mb * 32 + nl] : 0.0;
            const int64_t b_int = FP_EPI ? 0 : (int64_t)((u64)(int64_t)((const int *)bl)[wv * 64 + mb * 32 + nl] * ones);
#pragma unroll
            for (int c = 0; c < 4; c++) {
                double2 ts = make_double2(0.0, 0.0);
                if (POS7) ts = *(const double2 *)(tl + 16 * h + 8 * g + 2 * c);
#pragma unroll
                for (int e = 0; e < 2; e++) {
                    const int r = 8 * h + 2 * c + e;
                    if (FP_EPI) {
                        int S[PLANES];
#pragma unroll
                        for (int p = 0; p < PLANES; p++) S[p] = acc[p][mb][r];
                        res[c][e] = recombine_fp<PLANES, POS7>(S, POS7 ? b_fp - (e ? ts.y : ts.x) : b_fp, md);
                    } else {
                        int64_t t = b_int;
#pragma unroll
                        for (int p = 0; p < PLANES; p++) t += (int64_t)((u64)(int64_t)acc[p][mb][r] << (8 * p));
                        res[c][e] = reduce_signed(t, q, q_inv);
                    }
                }
            }
        };
        // A wave whose outputs do not exist has nothing to recombine, and in products of one output tile does not: 8 outputs of 32 to 512
        // operands 5 % of the kernel, 40 outputs 2 %.  (With more tiles it runs in step with the others: 825 outputs of 160
        // operands took 3 % longer where the last tile's three idle waves skipped.  Leaving out the second block of 32 as well takes
        // another 10 % at 8 outputs, and costs 1 to 4 % where all outputs exist.)
        if (n_tiles_m > 1 || i0 < m) {
            piece(0, 0);
#pragma unroll
            for (int mh = 0; mh < 4; mh++) {
                const int ib = i0 + (mh >> 1) * 32, h = mh & 1;
#pragma unroll
                for (int c = 0; c < 4; c++) *(ulonglong2 *)(o_lds + nl * AM_OROW + g * 64 + c * 16) = make_ulonglong2(res[c][0], res[c][1]);
                wave_lds_fence();
                ulonglong2 w[4];
#pragma unroll
                for (int k = 0; k < 4; k++) w[k] = *(const ulonglong2 *)(o_lds + (8 * k + (lane >> 3)) * AM_OROW + (lane & 7) * 16);
                if (mh < 3) piece((mh + 1) >> 1, (mh + 1) & 1);
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const int row = 8 * k + (lane >> 3);
                    const ct_pair v = {w[k].x, w[k].y};
                    u64 *o = out + (size_t)(ib + row) * ct_words_out + off_out + 16 * h + (lane & 7) * 2;
                    if (whole) *(ct_pair *)o = v;
                    else if (ib + row < m) *(ct_pair *)o = v;
                }
                wave_lds_fence();
            }
        }
        stores_pending = whole;
        if (!whole) wait_vmcnt<0>();  // some stores were left out: start the next item from a known count
        item = next;
    }
    wait_vmcnt<0>();  // no copy may still be in flight into LDS when the workgroup ends
}

// ---------------------------------------------------------------- few operands or few outputs: split and contraction in one kernel
// A block takes one word tile: the digits of its operands go straight to LDS (no planes in memory, no filling up to whole groups of steps)
// and each wave runs through blocks of 32 outputs.
//   CHUNKED = false: all operands fit LDS together (AMD_MAX_OPERANDS); a wave takes every fourth block of outputs.
//   CHUNKED = true:  one block of outputs a wave (AMD_MAX_OUTPUTS), which keeps its sums while the operands pass through LDS, AMD_CHUNK_STEPS
//   steps at a time.  Four waves, or eight over five planes, leave room for two blocks on a CU, so that one reads while the other multiplies; the others
//   read and multiply by turns.
// Bound by the reading of the operands and the writing of the outputs while the outputs are few, then by the fragment read from LDS that
// every matrix instruction needs (in k_accumulate_mfma every second one does).  Four waves for up to 128 outputs, eight for 256, twelve
// for 384: beyond that the sums do not fit the registers.
#define AMD_MAX_OPERANDS 384
#define AMD_MAX_OUTPUTS 384
#define AMD_CHUNKED_MIN 256  // operands from which they pass through LDS in chunks, where the outputs allow it: 300 and 8 outputs 0.20 -> 0.14 ms
                             // (2^14, 6 limbs), 300 and 256 0.38 -> 0.32; 200 and 256 0.22 -> 0.25
#define AMD_MAX_RESCALED 128  // operands that are rescaled on the way
#define AMD_CHUNK_STEPS 8
#define AM_LDS (160 << 10)  // of a CU
#define AMD_AHEAD 4  // steps whose words, or weights, are requested together
// RESCALE: the scalar-multiply + rescale step is applied to the operands on the way, as in k_byte_planes_rescale (fc: its constants); the limb that it
// drops is read and rescaled once for every limb that stays, which pays for few operands only.
template <int PLANES, int MODE, bool CHUNKED, int WAVES, bool RESCALE>
__global__ __launch_bounds__(64 * WAVES, WAVES == 12 ? 3 : 2) void k_accumulate_direct(const u64 *xbase, u32 xstride, int n_v, int nk, const v4i *wfrag, const void *bias,
                                                                     int m, int m_pad, AmPrimes pr, int N, int l1, int limb_stride_in, u64 *out,
                                                                     int limb_stride_out, const PrimeConst *pc, const double *fc) {
    HIP_DYNAMIC_SHARED(char, smem)
    static_assert(MODE != AM_POS7, "digits of 8 bits");
    constexpr bool FP_EPI = MODE != AM_INT8;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5, nl = lane & 31;
    const int steps = (n_v + AM_TILE_K - 1) / AM_TILE_K, cw = N / AM_TILE_N;
    const int pl = blockIdx.x / cw, poly = pl >= l1, limb = poly ? pl - l1 : pl, ctile = blockIdx.x - pl * cw;
    const u64 *xw = xbase + ((size_t)poly * limb_stride_in + limb) * N + (size_t)ctile * AM_TILE_N;
    // digits of steps s0 .. s1 - 1 to LDS, the first of them at step 0
    auto fill = [&](int s0, int s1) {
        constexpr int PARTS = WAVES / 4;  // steps that the block's threads take at a time
        const int k4 = tid >> 5 & 7, ln = tid & 31, part = wv >> 2;
        u32 *dst = (u32 *)smem + ((k4 >> 2) * 32 + plane_row(ln)) * 4 + (k4 & 3);
        AmFp mod, last;
        double k, k_q, qi, qi_q, kl, kl_q;
        const u64 *xl = xbase + ((size_t)poly * limb_stride_in + l1) * N + (size_t)ctile * AM_TILE_N;
        if (RESCALE) {
            const int lin = l1 + 1;
            mod = {(double)as_const(&pc[limb].q)[0], as_const(fc)[4 * lin + limb]};
            last = {(double)as_const(&pc[l1].q)[0], as_const(fc)[4 * lin + l1]};
            k = as_const(fc)[limb], k_q = as_const(fc)[lin + limb], qi = as_const(fc)[2 * lin + limb], qi_q = as_const(fc)[3 * lin + limb];
            kl = as_const(fc)[l1], kl_q = as_const(fc)[lin + l1];
        }
#pragma unroll 1
        for (int sa = s0 + part; sa < s1; sa += AMD_AHEAD * PARTS) {
            u64 w[AMD_AHEAD][4], wl[RESCALE ? AMD_AHEAD : 1][4];
#pragma unroll
            for (int s = 0; s < AMD_AHEAD; s++) {
                if (AMD_CHUNK_STEPS % (AMD_AHEAD * PARTS) && sa + s * PARTS >= s1) break;  // the next chunk's (read twice, 384 x 384 on 16 limbs of
                                                                                           // 2^16 took 4.97 ms, now 4.11; 2560 x 384 19.7, 18.7)
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    const int v = (sa + s * PARTS) * AM_TILE_K + 4 * k4 + j;
                    w[s][j] = v < n_v ? xw[(size_t)v * xstride + ln] : 0;
                    if (RESCALE) wl[s][j] = v < n_v ? xl[(size_t)v * xstride + ln] : 0;  // (no operand: zero stays zero)
                }
            }
            if (RESCALE) {
#pragma unroll
                for (int s = 0; s < AMD_AHEAD; s++)
#pragma unroll
                    for (int j = 0; j < 4; j++) {
                        const double c = last.mid(last.mulmod((double)wl[s][j], kl, kl_q));
                        const double t = mod.mulmod((double)w[s][j], k, k_q) - mod.mid(c);
                        const double r = mod.mid(mod.mulmod(mod.mid(t), qi, qi_q));
                        w[s][j] = (u64)(r < 0.0 ? r + mod.q : r);
                    }
            }
#pragma unroll
            for (int s = 0; s < AMD_AHEAD; s++) {
                if (sa + s * PARTS < s1) {
                    u32 d[8];
                    transpose4((u32)w[s][0], (u32)w[s][1], (u32)w[s][2], (u32)w[s][3], d);
                    transpose4((u32)(w[s][0] >> 32), (u32)(w[s][1] >> 32), (u32)(w[s][2] >> 32), (u32)(w[s][3] >> 32), d + 4);
#pragma unroll
                    for (int p = 0; p < PLANES; p++) dst[((sa + s * PARTS - s0) * PLANES + p) * 256] = d[p] ^ 0x80808080u;
                }
            }
        }
    };
    const char *planes = smem + lane * 16;
    // outputs ib .. ib + 31: adds the products of steps s0 .. s1 - 1, which lie in LDS from step 0 on
    auto contract = [&](v16i *acc, int ib, int s0, int s1) {
        const v4i *wp = wfrag + ((size_t)(ib / AM_TILE_M) * nk * 4 + ib % AM_TILE_M / 64) * 128 + ib % 64 / 32 * 64 + lane;
#pragma unroll 1
        for (int ka = s0; ka < s1; ka += AMD_AHEAD) {
            v4i wf[AMD_AHEAD];
#pragma unroll
            for (int s = 0; s < AMD_AHEAD; s++)
                if (ka + s < s1) wf[s] = wp[(size_t)(ka + s) * 512];
#pragma unroll
            for (int s = 0; s < AMD_AHEAD; s++) {
                if (ka + s < s1) {
#pragma unroll
                    for (int p = 0; p < PLANES; p++)
                        acc[p] = __builtin_amdgcn_mfma_i32_32x32x32_i8(*(const v4i *)(planes + ((ka + s - s0) * PLANES + p) * 1024), wf[s], acc[p], 0, 0, 0);
                }
            }
        }
    };
    char *o_lds = smem + (CHUNKED ? AMD_CHUNK_STEPS : steps) * PLANES * 1024 + wv * 32 * AM_OROW;
    const size_t ct_words_out = (size_t)2 * limb_stride_out * N;
    const size_t off_out = ((size_t)poly * limb_stride_out + limb) * N + (size_t)ctile * AM_TILE_N;
    const u64 q = pr.q[limb];
    const double q_inv = pr.q_inv[limb], qd = (double)q;
    const AmModulus md = {qd, q_inv, qd / AmDigits<false>::P4, q_inv * AmDigits<false>::P4};
    u64 ones = 0;
#pragma unroll
    for (int p = 0; p < PLANES; p++) ones |= (u64)1 << (8 * p);
    // the recombination and the stores as in k_accumulate_mfma: 32 outputs x 16 words at a time
    auto finish = [&](const v16i *acc, int ib) {
        double b_fp = 0.0;
        int64_t b_int = 0;
        if (FP_EPI) b_fp = ((const double *)bias)[(size_t)limb * m_pad + ib + nl];
        else b_int = (int64_t)((u64)(int64_t)((const int *)bias)[ib + nl] * ones);
#pragma unroll
        for (int h = 0; h < 2; h++) {
#pragma unroll
            for (int c = 0; c < 4; c++) {
                u64 res[2];
#pragma unroll
                for (int e = 0; e < 2; e++) {
                    const int r = 8 * h + 2 * c + e;
                    if (FP_EPI) {
                        int S[PLANES];
#pragma unroll
                        for (int p = 0; p < PLANES; p++) S[p] = acc[p][r];
                        res[e] = recombine_fp<PLANES, false>(S, b_fp, md);
                    } else {
                        int64_t t = b_int;
#pragma unroll
                        for (int p = 0; p < PLANES; p++) t += (int64_t)((u64)(int64_t)acc[p][r] << (8 * p));
                        res[e] = reduce_signed(t, q, q_inv);
                    }
                }
                *(ulonglong2 *)(o_lds + nl * AM_OROW + g * 64 + c * 16) = make_ulonglong2(res[0], res[1]);
            }
            wave_lds_fence();
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const int row = 8 * k + (lane >> 3);
                const ulonglong2 w = *(const ulonglong2 *)(o_lds + row * AM_OROW + (lane & 7) * 16);
                if (ib + row < m) *(ct_pair *)(out + (size_t)(ib + row) * ct_words_out + off_out + 16 * h + (lane & 7) * 2) = ct_pair{w.x, w.y};
            }
            wave_lds_fence();
        }
    };
    if (CHUNKED) {
        const int ib = wv * 32;
        v16i acc[PLANES] = {};
#pragma unroll 1
        for (int s0 = 0; s0 < steps; s0 += AMD_CHUNK_STEPS) {
            const int s1 = min(s0 + AMD_CHUNK_STEPS, steps);
            if (s0) __syncthreads();  // every wave has read the chunk before
            fill(s0, s1);
            __syncthreads();
            if (ib < m) contract(acc, ib, s0, s1);
        }
        if (ib < m) finish(acc, ib);
    } else {
        fill(0, steps);
        __syncthreads();
#pragma unroll 1
        for (int ib = wv * 32; ib < m; ib += 32 * WAVES) {
            v16i acc[PLANES] = {};
            contract(acc, ib, 0, steps);
            finish(acc, ib);
        }
    }
}

static bool amd_chunked(int n_v, int m) { return n_v > AMD_CHUNKED_MIN && m <= AMD_MAX_OUTPUTS; }
// LDS of a block: the digits of `steps` steps and each wave's results.
static constexpr int amd_lds(int planes, int steps, int waves) { return steps * planes * 1024 + waves * 32 * AM_OROW; }

// Whether a product of n_v operands and m outputs over `tiles` word tiles takes the kernel above.  The other way keeps planes in memory, split for
// whole groups of 256 operands, and contracts them for whole tiles of 256 outputs, item by item on all CUs.  Whole calls, this way over that one (the lower
// the better), on 2 limbs of the 2^10 ring (128 tiles), 3 of 2^11 (384), 3 of 2^12 (768), 6 of 2^14 (6144) and 16 of 2^16 (65536), primes of 50 bits:
//   operands x outputs   64 x 8 .38 .25 .19 .15 .15      64 x 512 .74 .56 .48 .48 .55      64 x 4096 1.32 .83 .60 .53 .50
//                        256 x 8 .50 .32 .51 .43 .42     256 x 1024 1.36 .82 .82 .71 .78   256 x 4096 1.95 1.03 1.00 .84 .84
//                        384 x 384 .70 .73 .64 .59 .69   384 x 1024 1.42 1.25 .94 .91 .94  384 x 4096 1.86 1.32 .93 .93 1.06
//                        1024 x 8 .83 .46 .47 .38 .41    1024 x 384 1.00 .83 .60 .63 .64   4096 x 384 1.06 .75 .62 .61
// A block runs through all outputs of its word tile: what costs is CUs that have no block, or none in the last round, as long as that takes.  m times the idle
// share of the rounds is a measure of it.
//   - Few outputs (a block of 32 a wave): as many tiles as three quarters of the CUs, or few enough operands.
//   - All operands in LDS, fewer tiles than CUs: up to 480 idle outputs (16 x 1024, 128 tiles: .83; 128 x 1024: 1.04), of more than 128 operands 192
//     (384 x 768, 192 tiles: .92; 384 x 1024: 1.10) or 384 outputs in all.  With as many tiles as CUs: up to 128 operands always;
//     two blocks to a CU: up to 512 idle outputs, 640 where the planes take a second group of operands (256 x 2048, 640 tiles: .95; 256 x 4096: 1.05);
//     one block to a CU: up to 64 (257 x 1024, 576 tiles: 1.12; 257 x 640: .97), and up to 1.4 million weights (6 limbs of 2^14: 384 x 3072 .92, 350 x 4096
//     .94, 384 x 4096 .97, 257 x 6144 1.03, 384 x 6144 1.14; 16 of 2^16: .98, 1.02, 1.05, 1.01, 1.10).
//   - With the rescale: up to 128 operands as above (16 limbs of 2^16, 128 x 512 .90, 128 x 4096 .74; 200 x 200 1.13).
// Its digits are of 8 bits and its weights signed: weights prepared for the digits of AM_POS7 are not for it, whatever the sizes.
bool am_direct(int n_cu, int tiles, int planes, int mode, int n_v, int m, bool rescale) {
    if (mode == AM_POS7 || (rescale && n_v > AMD_MAX_RESCALED)) return false;
    if (amd_chunked(n_v, m)) return 4l * tiles >= 3l * n_cu || n_v <= 512 + 2 * tiles;
    if (n_v > AMD_MAX_OPERANDS) return false;
    const auto idle = [&](int places, long outputs) {  // whether the places of the last round that are empty would have done more than `outputs`
        const long all = (long)((tiles + places - 1) / places) * places;
        return m * (all - tiles) > outputs * all;
    };
    if (n_v <= 128) return tiles >= n_cu || !idle(n_cu, 480);
    if (tiles < n_cu) return m <= AMD_MAX_OUTPUTS || !idle(n_cu, 192);
    if (2 * amd_lds(planes, (n_v + AM_TILE_K - 1) / AM_TILE_K, 4) <= AM_LDS) return !idle(2 * n_cu, n_v > 256 ? 640 : 512);
    return !idle(n_cu, 64) && (long)n_v * m <= 1400000;
}

template <int P, int MODE>
static void am_launch_direct(ensi_ctx *ctx, hipStream_t st, const u64 *xbase, u32 xstride, int n_v, int n_kpad, const v4i *wfrag, const void *bias, int m,
                             int l1, int limb_stride_in, u64 *out, int limb_stride_out, int n_tiles_m, const double *d_rescale) {
    AmPrimes pr;
    for (int i = 0; i < ENSI_MAX_EXT; i++) {
        pr.q[i] = i < l1 ? ctx->primes[i] : 1;
        pr.q_inv[i] = 1.0 / (double)pr.q[i];
    }
    const int steps = (n_v + AM_TILE_K - 1) / AM_TILE_K;
    ScopedTimer t(ctx, d_rescale ? "rescale_accumulate_direct" : "accumulate_direct", st);
    auto launch = [&](auto chunked, auto waves, auto rescale) {
        constexpr bool CHUNKED = decltype(chunked)::value, RESCALE = decltype(rescale)::value;
        constexpr int WAVES = decltype(waves)::value;
        auto lds = [](int s) { return amd_lds(P, s, WAVES); };
        bool &attr_set = ctx->am_direct_attr_set[((2 * MODE + (P == 5 ? 0 : 1)) * 4 + (CHUNKED ? WAVES / 4 : 0)) * 2 + RESCALE];
        if (!attr_set) {
            (void)hipFuncSetAttribute((const void *)k_accumulate_direct<P, MODE, CHUNKED, WAVES, RESCALE>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                      lds(CHUNKED ? AMD_CHUNK_STEPS : AMD_MAX_OPERANDS / AM_TILE_K));
            attr_set = true;
        }
        hipLaunchKernelGGL((k_accumulate_direct<P, MODE, CHUNKED, WAVES, RESCALE>), dim3(2 * l1 * (ctx->N / AM_TILE_N)), dim3(64 * WAVES),
                           lds(CHUNKED ? AMD_CHUNK_STEPS : steps), st, xbase, xstride, n_v, n_kpad / AM_TILE_K, wfrag, bias, m, n_tiles_m * AM_TILE_M, pr, ctx->N,
                           l1, limb_stride_in, out, limb_stride_out, ctx->d_pc, d_rescale);
    };
    typedef std::integral_constant<int, 4> Four;
    typedef std::integral_constant<int, 8> Eight;
    typedef std::integral_constant<int, 12> Twelve;
    typedef std::false_type No;
    typedef std::true_type Yes;
    if (d_rescale) {
        if constexpr (MODE == AM_FP8) launch(No(), Four(), Yes());  // (the only mode that comes here with a rescale)
    } else if (!amd_chunked(n_v, m))
        launch(No(), Four(), No());
    else if (m <= 128)
        launch(Yes(), Four(), No());
    else if (m <= 256)
        launch(Yes(), Eight(), No());
    else
        launch(Yes(), Twelve(), No());
}

template <int P, int MODE>
static void am_launch(ensi_ctx *ctx, unsigned grid, hipStream_t st, const u64 *xbase, u32 xstride, int n_v, int n_kpad, const v4i *wfrag,
                      const void *bias, int m, int l1, int limb_stride_in, u64 *out, int limb_stride_out, int n_tiles_m, int workers,
                      int m_group, char *xp, int slice_ctiles, const double *d_rescale) {
    constexpr bool POS7 = MODE == AM_POS7;
    bool &attr_set = ctx->am_attr_set[2 * MODE + (P == 5 ? 0 : 1)];
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void *)k_accumulate_mfma<P, MODE>, hipFuncAttributeMaxDynamicSharedMemorySize, AmLayout<P>::total);
        attr_set = true;
    }
    const int nk = n_kpad / AM_TILE_K, ctiles = ctx->N / AM_TILE_N;
    AmPrimes pr;
    for (int i = 0; i < ENSI_MAX_EXT; i++) {
        pr.q[i] = i < l1 ? ctx->primes[i] : 1;
        pr.q_inv[i] = 1.0 / (double)pr.q[i];
    }
    // behind the planes of a slice: its partial word sums, then the word sums
    const int parts = d_rescale ? nk / AM_RS_STEPS : nk / 8;
    u64 *part = (u64 *)(xp + (size_t)2 * l1 * slice_ctiles * nk * P * 1024);
    double *tsum = (double *)(part + (size_t)2 * l1 * slice_ctiles * parts * AM_TILE_N);
    for (int c0 = 0; c0 < ctiles; c0 += slice_ctiles) {
        const int cw = std::min(slice_ctiles, ctiles - c0), n_words = 2 * l1 * cw * AM_TILE_N;
        {
            ScopedTimer t(ctx, d_rescale ? "rescale_byte_planes" : "byte_planes", st);
            if (d_rescale)
                hipLaunchKernelGGL((k_byte_planes_rescale<P, POS7>), dim3(cw, nk / AM_RS_STEPS, 2), dim3(AM_THREADS), 0, st, xbase, xstride, n_v, nk, ctx->N, l1,
                                   limb_stride_in, c0, cw, xp, ctx->d_pc, d_rescale, part);
            else
                hipLaunchKernelGGL((k_byte_planes<P, POS7>), dim3(cw, nk / 8, 2 * l1), dim3(AM_THREADS), 0, st, xbase, xstride, n_v, nk, ctx->N, l1,
                                   limb_stride_in, c0, cw, xp, part);
        }
        if (POS7) {
            ScopedTimer t(ctx, "word_sums", st);
            hipLaunchKernelGGL(k_word_sums, dim3((n_words + AM_THREADS - 1) / AM_THREADS), dim3(AM_THREADS), 0, st, part, parts, n_words, cw, l1, ctx->d_pc, tsum);
        }
        {
            ScopedTimer t(ctx, "accumulate_mfma", st);
            hipLaunchKernelGGL((k_accumulate_mfma<P, MODE>), dim3(grid), dim3(AM_THREADS), AmLayout<P>::total, st, (const char *)xp, c0, cw, n_kpad, wfrag,
                               bias, tsum, m, pr, ctx->N, l1, out, limb_stride_out, 2 * l1 * cw, n_tiles_m, workers, m_group);
        }
    }
}

// Coefficient tiles per slice: all of them if their planes fit the budget.
static int am_slice_ctiles(int ctiles, int l1, int n_kpad, int planes) {
    const size_t per_ctile = (size_t)2 * l1 * (n_kpad / AM_TILE_K) * (planes <= 5 ? 5 : 7) * 1024;
    const size_t budget = (size_t)16 << 30;
    return (int)std::min<size_t>((size_t)ctiles, std::max<size_t>(budget / per_ctile, 1));
}

// d_rescale != nullptr: the operands are read at l1 + 1 limbs and the scalar-multiply + rescale step is applied while
// their planes are built (constants as for k_rescale_fp at l1 + 1 limbs); out is at l1 limbs.
int launch_accumulate_mfma(ensi_ctx *ctx, const u64 *xbase, size_t xstride, int n_v, int n_kpad, const int8_t *d_wt, const int32_t *d_bias,
                           const double *d_bias_fp, int planes, int mode, int m, int l1, int limb_stride_in, u64 *out, int limb_stride_out, const double *d_rescale,
                           hipStream_t st) {
    if (d_rescale && mode == AM_INT8) {  // (the rescale on the way works in double precision)
        ctx->err = "the rescale is fused with the signed sums for primes below 2^50 only";
        return ENSI_E_BADARG;
    }
    const int ctiles = ctx->N / AM_TILE_N;
    const int n_tiles_m = (m + AM_TILE_M - 1) / AM_TILE_M;
    int &n_cu = ctx->n_cu;
    if (!n_cu) {
        hipDeviceProp_t prop;
        n_cu = hipGetDeviceProperties(&prop, ctx->device) == hipSuccess ? prop.multiProcessorCount : 256;
        if (n_cu < 8) n_cu = 8;
    }
    const int workers = n_cu / 8;  // one persistent workgroup per CU; workgroup b runs on XCD b % 8
    const unsigned grid = 8u * (unsigned)workers;
    const v4i *wf = (const v4i *)d_wt;
    const int m_group = 8;  // 8 output tiles x 4 word tiles in flight per XCD
    const int P = planes <= 5 ? 5 : 7;
    const void *bias = mode == AM_INT8 ? (const void *)d_bias : (const void *)d_bias_fp;
    if (am_direct(n_cu, 2 * l1 * ctiles, P, mode, n_v, m, d_rescale != nullptr)) {
#define AMD_LAUNCH(PL, MODE) \
    am_launch_direct<PL, MODE>(ctx, st, xbase, (u32)xstride, n_v, n_kpad, wf, bias, m, l1, limb_stride_in, out, limb_stride_out, n_tiles_m, d_rescale)
        if (mode == AM_INT8) AMD_LAUNCH(7, AM_INT8);
        else if (P == 5) AMD_LAUNCH(5, AM_FP8);
        else AMD_LAUNCH(7, AM_FP8);
#undef AMD_LAUNCH
        return ENSI_OK;
    }
    const int slice_ctiles = am_slice_ctiles(ctiles, l1, n_kpad, P);
    const size_t tiles = (size_t)slice_ctiles * 2 * l1, nk = n_kpad / AM_TILE_K;
    const size_t xp_words = tiles * nk * P * 128 + (mode == AM_POS7 ? tiles * (nk / AM_RS_STEPS + 1) * AM_TILE_N : 0);
    if (ctx->ws_xp_words < xp_words) {
        if (ctx->ws_xp) (void)hipFree(ctx->ws_xp);
        ctx->ws_xp = nullptr;
        ctx->ws_xp_words = 0;
        if (ctx->pool->alloc((void **)&ctx->ws_xp, xp_words * 8) != hipSuccess) {
            ctx->err = "device allocation of the byte-plane workspace failed";
            return ENSI_E_NOMEM;
        }
        ctx->ws_xp_words = xp_words;
    }
#define AM_LAUNCH(PL, MODE)                                                                                                              \
    am_launch<PL, MODE>(ctx, grid, st, xbase, (u32)xstride, n_v, n_kpad, wf, bias, m, l1, limb_stride_in, out, limb_stride_out, n_tiles_m, \
                        workers, m_group, (char *)ctx->ws_xp, slice_ctiles, d_rescale)
    if (mode == AM_POS7) {
        if (P == 5) AM_LAUNCH(5, AM_POS7);
        else AM_LAUNCH(7, AM_POS7);
    } else if (mode == AM_FP8) {
        if (P == 5) AM_LAUNCH(5, AM_FP8);
        else AM_LAUNCH(7, AM_FP8);
    } else {
        AM_LAUNCH(7, AM_INT8);
    }
#undef AM_LAUNCH
    return ENSI_OK;
}

// ---------------------------------------------------------------- sustained rate of the matrix instruction
// A register-only loop of V_MFMA_I32_32X32X32_I8 on the digits and weights that the contraction has at the context's primes
// (the clock the chip holds hangs on them), one accumulator block per plane, one workgroup of four waves per CU like the
// contraction: what the matrix pipes deliver at the clock the chip holds under that load.  No memory is touched inside
// the loop; the operands come from `seed` so that the compiler cannot fold the loop: [planes][1024] words of digits, then
// RATE_WEIGHTS vectors of 1024 words of weights, taken in turn as an output's weights change from step to step.
#define RATE_PLANES 7
#define RATE_WEIGHTS 2
__global__ __launch_bounds__(AM_THREADS) void k_matrix_rate(const v4i *seed, int iters, int *sink) {
    v4i a[RATE_PLANES], b[RATE_WEIGHTS];
#pragma unroll
    for (int p = 0; p < RATE_PLANES; p++) a[p] = seed[p * AM_THREADS + threadIdx.x];
#pragma unroll
    for (int w = 0; w < RATE_WEIGHTS; w++) b[w] = seed[(RATE_PLANES + w) * AM_THREADS + threadIdx.x];
    v16i d[RATE_PLANES];
#pragma unroll
    for (int p = 0; p < RATE_PLANES; p++)
#pragma unroll
        for (int r = 0; r < 16; r++) d[p][r] = 0;
    for (int it = 0; it < iters; it++) {
#pragma unroll
        for (int w = 0; w < RATE_WEIGHTS; w++)
#pragma unroll
            for (int p = 0; p < RATE_PLANES; p++) d[p] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[p], b[w], d[p], 0, 0, 0);
    }
    int t = 0;
#pragma unroll
    for (int p = 0; p < RATE_PLANES; p++) t += d[p][p];
    if (t == 0x7fffffff) sink[0] = t;  // keeps the loop alive; never true for these operands in practice, harmless if it is
}

int launch_matrix_rate(ensi_ctx *ctx, double seconds, double *ops_per_second, hipStream_t st) {
    int &n_cu = ctx->n_cu;
    if (!n_cu) {
        hipDeviceProp_t prop;
        n_cu = hipGetDeviceProperties(&prop, ctx->device) == hipSuccess ? prop.multiProcessorCount : 256;
        if (n_cu < 8) n_cu = 8;
    }
    int qbits = 0;
    for (int i = 0; i < ctx->L; i++) qbits = std::max(qbits, 64 - __builtin_clzll(ctx->primes[i]));
    const bool pos7 = am_pos7_primes(qbits);
    const size_t plane = (size_t)AM_THREADS * sizeof(v4i), n_digits = RATE_PLANES * plane, n_weights = RATE_WEIGHTS * plane;
    std::vector<int8_t> h(n_digits + n_weights);
    u64 x = 0x9E3779B97F4A7C15ull;
    for (size_t k = 0; k < h.size(); k++) {
        x = x * 6364136223846793005ull + 1442695040888963407ull;
        const u32 r = (u32)(x >> 32);
        if (k < n_digits) {
            h[k] = (int8_t)(pos7 && k / plane < RATE_PLANES - 1 ? r >> 25 : r >> 24);
        } else {
            const int w = r < 1288490189u ? -1 : r < 3006477107u ? 0 : 1;  // 3 : 4 : 3
            h[k] = (int8_t)(pos7 ? w + 1 : w);
        }
    }
    v4i *d_seed = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipError_t e = ctx->pool->alloc((void **)&d_seed, h.size() + sizeof(int));
    if (e == hipSuccess) e = hipMemcpy(d_seed, h.data(), h.size(), hipMemcpyHostToDevice);
    int *sink = (int *)((char *)d_seed + h.size());
    if (e == hipSuccess) e = hipEventCreate(&e0);
    if (e == hipSuccess) e = hipEventCreate(&e1);
    float ms = 0;
    // about 32 pipe cycles per instruction at roughly 1.6 GHz; the measured time is what counts
    const int iters = (int)std::max(1000.0, seconds * 1.6e9 / (32.0 * RATE_PLANES * RATE_WEIGHTS));
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_matrix_rate, dim3(n_cu), dim3(AM_THREADS), 0, st, d_seed, 1000, sink);
        (void)hipEventRecord(e0, st);
        hipLaunchKernelGGL(k_matrix_rate, dim3(n_cu), dim3(AM_THREADS), 0, st, d_seed, iters, sink);
        (void)hipEventRecord(e1, st);
        e = hipEventSynchronize(e1);
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (d_seed) (void)hipFree(d_seed);
    if (e != hipSuccess || !(ms > 0)) {
        ctx->err = "the matrix-rate probe failed";
        return ENSI_E_HIP;
    }
    const double n_inst = (double)n_cu * 4 * (double)iters * RATE_PLANES * RATE_WEIGHTS;
    *ops_per_second = n_inst * 2.0 * 32 * 32 * 32 / (ms * 1e-3);
    return ENSI_OK;
}
