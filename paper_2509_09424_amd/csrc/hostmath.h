// Host-side exact modular helpers (context set-up only; never on the hot path).
#pragma once
#include <stdint.h>

#include "modarith.h"

static inline u64 hm_mulmod(u64 a, u64 b, u64 q) { return (u64)(((u128)a * b) % q); }
static inline u64 hm_powmod(u64 a, u64 e, u64 q) {
    u64 r = 1 % q;
    a %= q;
    while (e) {
        if (e & 1) r = hm_mulmod(r, a, q);
        a = hm_mulmod(a, a, q);
        e >>= 1;
    }
    return r;
}
// q prime
static inline u64 hm_invmod(u64 a, u64 q) { return hm_powmod(a, q - 2, q); }
// floor(w * 2^64 / q), w < q
static inline u64 hm_shoup(u64 w, u64 q) { return (u64)((((u128)w) << 64) / q); }
// w * 2^64 mod q
static inline u64 hm_to_mont(u64 w, u64 q) { return (u64)((((u128)w) << 64) % q); }
// -q^{-1} mod 2^64, q odd (Newton iteration)
static inline u64 hm_neg_inv64(u64 q) {
    u64 x = q;  // correct to 3 bits
    for (int i = 0; i < 6; i++) x *= 2 - q * x;
    return (u64)0 - x;
}
// Two int32 halves of v packed into one word, v = high * 2^bits + low with low in [-2^(bits-1), 2^(bits-1)] (slightly
// beyond where the high half would leave 31 bits).
static inline u64 hm_split(int64_t v, int bits) {
    int64_t hi = (v + ((int64_t)1 << (bits - 1))) >> bits;
    if (hi > 0x7fffffff) hi = 0x7fffffff;
    const int64_t lo = v - hi * ((int64_t)1 << bits);
    return ((u64)(u32)(int32_t)hi << 32) | (u32)(int32_t)lo;
}
static inline int64_t hm_centred(u64 w, u64 q) { return w > q / 2 ? (int64_t)w - (int64_t)q : (int64_t)w; }
// Primes of the PRIME_WIDE arithmetic (ArithWide, whose bounds need this d).
static constexpr u64 HM_WIDE_D = (u64)1 << 26;
static inline bool hm_is_wide(u64 q) { return q < ((u64)1 << 60) && q > ((u64)1 << 60) - HM_WIDE_D; }
// multiplier of the PRIME_WIDE arithmetic: the centred residue, split at 28 bits
static inline u64 hm_wide_pack(u64 w, u64 q) { return hm_split(hm_centred(w, q), 28); }
static inline bool hm_is_prime(u64 n) {
    if (n < 2) return false;
    static const u64 bases[] = {2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37};
    for (u64 b : bases) {
        if (n % b == 0) return n == b;
    }
    u64 d = n - 1;
    int r = 0;
    while ((d & 1) == 0) {
        d >>= 1;
        r++;
    }
    for (u64 b : bases) {
        u64 y = hm_powmod(b, d, n);
        if (y == 1 || y == n - 1) continue;
        bool comp = true;
        for (int i = 1; i < r; i++) {
            y = hm_mulmod(y, y, n);
            if (y == n - 1) {
                comp = false;
                break;
            }
        }
        if (comp) return false;
    }
    return true;
}
