// Small host-side helpers shared by the translation units that hold the C ABI.
#pragma once
#include <algorithm>
#include <vector>

#include "common.h"
// ------------------------------------------------------------------ utilities

struct DevBuf {
    void *p = nullptr;
    DevBuf() {}
    DevBuf(const DevBuf &) = delete;
    ~DevBuf() {
        if (p) (void)hipFree(p);
    }
    hipError_t alloc(ensi_ctx *ctx, size_t bytes) { return ctx->pool->alloc(&p, bytes ? bytes : 8); }
    template <class T>
    T *as() { return (T *)p; }
};

// The same for memory that the next call of its kind wants again: kept by the pool in between (allocating and freeing 16 MiB takes
// 0.3 ms).  Taking it waits for the device where a kept block serves, giving it back waits for nothing.
struct KeptBuf {
    DevPool *pool = nullptr;
    void *p = nullptr;
    size_t bytes = 0;
    KeptBuf() {}
    KeptBuf(const KeptBuf &) = delete;
    ~KeptBuf() {
        if (p) pool->give(p, bytes);
    }
    hipError_t take(ensi_ctx *ctx, size_t n) {
        pool = ctx->pool.get();
        return pool->take(&p, n, &bytes);
    }
};

template <class T>
inline hipError_t upload(ensi_ctx *ctx, T **d, const std::vector<T> &h) {
    hipError_t e = ctx->pool->alloc((void **)d, std::max<size_t>(h.size() * sizeof(T), 8));
    if (e != hipSuccess) return e;
    return hipMemcpy(*d, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice);
}

inline LimbMap make_map(const ensi_ctx *ctx, int l1, bool with_p) {
    LimbMap m;
    m.n = l1 + (with_p ? ctx->K : 0);
    for (int e = 0; e < ENSI_MAX_EXT; e++) m.prime[e] = 0;
    for (int e = 0; e < m.n; e++) m.prime[e] = e < l1 ? e : ctx->L + (e - l1);
    return m;
}

inline u32 galois_element(const ensi_ctx *ctx, int32_t step) {
    const int n = ctx->N / 2;
    int k = step % n;
    if (k < 0) k += n;
    return ctx->rot_exp[k];
}
inline u32 inv_mod_2n(u32 g, int N) {
    // g odd: Newton iteration modulo a power of two
    u32 x = g;
    for (int i = 0; i < 5; i++) x *= 2 - g * x;
    return x & (2 * (u32)N - 1);
}

inline int grow(ensi_ctx *ctx, u64 **p, size_t *have, size_t need) {
    if (*have >= need) return ENSI_OK;
    if (*p) ENSI_HIP(ctx, hipFree(*p));
    *p = nullptr;
    *have = 0;
    hipError_t e = ctx->pool->alloc((void **)p, need * sizeof(u64));
    if (e != hipSuccess) ENSI_FAIL(ctx, ENSI_E_NOMEM, "device allocation of %zu bytes failed: %s", need * sizeof(u64), hipGetErrorString(e));
    *have = need;
    return ENSI_OK;
}



// The library's own sampler of small polynomials (api_keys.hip): operating-system randomness when the context's
// seed is 0, a deterministic test generator otherwise.  Return an ENSI_E_* code.
int sample_ternary(ensi_ctx *ctx, int8_t *out, size_t n);
int sample_error(ensi_ctx *ctx, int8_t *out, size_t n);

// dst (device) <- src (host, any memory) on the stream: returns at once, never waits for the stream, and src may be reused or freed as soon as the
// call returns.  Up to UPLOAD_BYTES of whole words travel as a kernel's arguments, the rest through the context's ring of pinned buffers.
#define UPLOAD_BYTES 3072
hipError_t host_to_device(ensi_ctx *ctx, void *dst, const void *src, size_t bytes, hipStream_t st);

// ---- key switching, shared by the entry points (api.hip) -------------------------------------------------
// Intermediates of a batch of key switches: raised digits (raised_words per ciphertext), accumulators
// (2 (l1+K) N words per rotation).
struct KsWorkspace {
    u64 *digits, *u;
};
// Whether each raised ciphertext serves few rotations (RAISE_ONE: the fused path leaves its digits after their column pass, and the
// inner product runs their row passes, once per rotation) or many (their row passes are run once, by a kernel of their own).
enum RaiseUse { RAISE_ONE, RAISE_SHARED };
// A row pass of its own takes the digits through memory twice more; one in the inner product costs arithmetic that the reads of keys
// partly hide, and the digits of neighbouring rotations come from L2.  Two rotations a raise: 96 ciphertexts
// under Alg. 2 at 16 + 4 limbs 14.0 -> 12.6 ms; one: 64 columns of scores 90.7 -> 86.6; three: nothing in it (86.2, and 1152 rotations
// of the 2^14 ring in 7.26 against 7.24).  On every ring and for every kind of special primes: inner product and row pass of two
// rotations a raise, in column form against rows, 0.98 and 1.22 ms (just below 2^60), 1.21 and 1.32 (others above 2^50), 1.07 and 1.20
// (below 2^50) on 2^16; 0.245 and 0.288, 0.303 and 0.325, 0.273 and 0.282 on 2^14; 0.117 and 0.131, 0.145 and 0.158, 0.128 and 0.123
// (the one that loses) on 2^13.  The row pass runs over everything that was raised, so it is the average that counts: one
// of 32 inputs with 63 rotations, the others with none, 0.137 against 0.116 + 0.048 on 2^14.
// Rotations in groups (members > 1: their inner products are added before one inverse pass) read transformed digits only.
#define RAISE_ONE_MAX 2  // rotations per raise
inline RaiseUse raise_use(size_t n_rot, size_t n_raised, int members = 1) {
    return members == 1 && n_rot <= RAISE_ONE_MAX * n_raised ? RAISE_ONE : RAISE_SHARED;
}
size_t raised_words(const ensi_ctx *ctx, int l1);
int get_modup(ensi_ctx *ctx, int l1, const ModUpConst **out);
int get_moddown(ensi_ctx *ctx, int l1, const ModDownConst **out);
int get_ks16(ensi_ctx *ctx, int l1, const Ks16Const **out);
int raise_cts(ensi_ctx *ctx, int l1, const u64 *ct_base, size_t ct_stride_words, int limb_stride, int n_ct, RaiseUse use, hipStream_t st,
              const KsWorkspace *ws = nullptr);
int run_rotations(ensi_ctx *ctx, const RotDesc *d_desc, int n_rot, int l1, int limb_stride_in, int limb_stride_out, RaiseUse use, hipStream_t st,
                  int members = 1, const RotDesc *h_desc = nullptr, const KsWorkspace *ws = nullptr);

// Resolves the device address of the statically linked workspace for the context's device (api_static.hip).
int ensi_static_init(ensi_ctx *ctx);
// Allocates every slot of the staging ring and its event now, so that later small uploads allocate nothing.
int stage_prealloc(ensi_ctx *ctx);

// ---- helpers defined in one translation unit of the C ABI and used by others ---------------------------------
// api.hip
int encode_window(ensi_ctx *ctx, const double *slots, int n_pt, int n_slots, int slot0, int slot_step, int limbs, double scale,
                  ensi_pt **out);
int rot_chunk(const ensi_ctx *ctx);        // ciphertexts per group of a batched rotation
int ensure_desc(ensi_ctx *ctx, size_t n);  // grows the context's descriptor table to n entries
// api_matmul.hip
void free_plan(MatmulPlan *p);
// Constants of the scalar-multiply + rescale step at l1 limbs (integer set and fp64 set), uploaded to the context's
// small-constants workspace; kr = the integer the limbs are multiplied by before the division (1: plain rescale).
int upload_rescale_consts(ensi_ctx *ctx, int l1, double kr, bool negative, hipStream_t st, const u64 **d_consts, const double **d_fconsts,
                          bool *fp_out);
// api_pmult.hip: out_o = Rescale(sum of the terms [begin[o], begin[o+1]) of src (x) plaintext)
int pmult_core(ensi_ctx *ctx, const std::vector<PmTerm> &terms_in, const std::vector<int32_t> &begin, int l1, int limb_stride_in,
               const ensi_pt *pt, ensi_ct *out, hipStream_t st);
