"""GPU parity: the HIP library against the CPU oracle, through the C ABI, on the
same seeded inputs.  Integer results (RNS limbs) must match bit for bit;
decrypted slots must lie within 1e-3 of the float64 product."""
import numpy as np
import pytest

import workloads as wl
from helpers import Pair, stack_cts, to_oracle_cts

pytestmark = pytest.mark.gpu

TINY = wl.WORKLOADS[0].param_tuple()
# a small ring with the BitNet-shaped workloads' chain structure (alpha=4, partial last digit at lower levels)
SMALL4 = (10, 50, 6, 60, 4, 4, 40)
SMALL3 = (10, 50, 5, 60, 3, 3, 40)  # alpha=3: digits 3+2


@pytest.fixture(scope="module")
def tiny():
    p = Pair(TINY)
    yield p
    p.close()


@pytest.fixture(scope="module")
def small4():
    p = Pair(SMALL4)
    yield p
    p.close()


def test_primes_match_oracle(tiny):
    q, p = tiny.ctx.primes()
    assert q == tiny.pr.q and p == tiny.pr.p


def test_ntt_roundtrip_and_evaluation_set(tiny):
    rng = np.random.default_rng(0)
    primes = tiny.pr.q + tiny.pr.p
    x = np.stack([rng.integers(0, m, size=tiny.N, dtype=np.uint64) for m in primes])
    # ship the rows to the device inside a ciphertext-shaped import (2 ciphertexts x 2 polys x 1 limb)
    ct = tiny.ctx.ct_import(x.reshape(2, 2, 1, tiny.N) % np.uint64(tiny.pr.q[0]), 1.0)
    x = ct.export().reshape(4, tiny.N)
    idx = [0, 0, 0, 0]
    tiny.ctx.ntt(ct.device_ptr, idx, inverse=False)
    fwd = ct.export().reshape(4, tiny.N)
    want = tiny.o.ntt(x, [tiny.pr.q[0]] * 4)
    # whichever primitive root a side picked, the transform is the set of evaluations at all odd powers
    assert np.array_equal(np.sort(fwd, axis=1), np.sort(want, axis=1))
    assert not np.array_equal(fwd, x)
    tiny.ctx.ntt(ct.device_ptr, idx, inverse=True)
    assert np.array_equal(ct.export().reshape(4, tiny.N), x)
    ct.free()


def test_encode_within_one_and_import_export(tiny):
    rng = np.random.default_rng(1)
    z = rng.uniform(-1, 1, (2, tiny.n))
    pt = tiny.ctx.encode(z, tiny.pr.L)
    got = tiny.ctx.pt_export(pt)
    want = np.stack([tiny.o.encode_coeffs(v) for v in z])
    assert np.abs(got - want).max() <= 1
    assert (got != want).mean() < 0.01
    pt2 = tiny.ctx.pt_import(want, tiny.pr.L)
    assert np.array_equal(tiny.ctx.pt_export(pt2), want)
    pt.free()
    pt2.free()


def test_encrypt_bit_exact_and_decrypt(tiny):
    rng = np.random.default_rng(2)
    z = rng.uniform(-1, 1, (3, tiny.n))
    o_cts, g_ct = tiny.encrypt_both(z, tiny.pr.L)
    assert np.array_equal(g_ct.export(), stack_cts(o_cts))
    got = tiny.ctx.decrypt(tiny.g_sk, g_ct)
    want = np.stack([tiny.o.decrypt(c, tiny.o_sk) for c in o_cts])
    assert np.abs(got - want).max() < 1e-7
    assert np.abs(got - z).max() < 1e-3
    part = tiny.ctx.decrypt(tiny.g_sk, g_ct, slot_begin=64, n_slots=32)
    assert np.abs(part - want[:, 64:96]).max() < 1e-7
    g_ct.free()


@pytest.mark.parametrize("params", [TINY, SMALL4, SMALL3], ids=["tiny", "alpha4", "alpha3"])
def test_rotate_bit_exact(params):
    p = Pair(params)
    try:
        steps = [1, -1, 5, p.n // 2, 3]
        o_gks, g_gk = p.galois_keys(sorted(set(steps)))
        z = p.rng.uniform(-1, 1, (len(steps), p.n))
        for limbs in sorted({p.pr.L, max(2, p.pr.L - 1), 2}, reverse=True):
            o_cts, g_ct = p.encrypt_both(z, limbs)
            out = p.ctx.rotate(g_gk, g_ct, steps)
            want = [p.o.rotate(c, o_gks[st]) for c, st in zip(o_cts, steps)]
            assert np.array_equal(out.export(), stack_cts(want)), "limbs=%d" % limbs
            dec = p.ctx.decrypt(p.g_sk, out)
            for i, st in enumerate(steps):
                assert np.abs(dec[i] - np.roll(z[i], -st)).max() < 1e-3
            assert out.limbs == limbs and out.scale == g_ct.scale
            out.free()
            g_ct.free()
        g_gk.free()
    finally:
        p.close()


@pytest.mark.parametrize("placement", ["diagonal", "zero"])
def test_tiny_workload_matmul_bit_exact(tiny, placement):
    w = wl.WORKLOADS[0]
    rng = wl.rng_for(w.index)
    W = wl.ternary_weights(rng, w.d_in, w.d_out)
    X = wl.activations(rng, w.tokens, w.d_in, w.act)
    packed = wl.pack_columns(X, tiny.n)
    o_cts, g_ct = tiny.encrypt_both(packed, tiny.pr.L)
    rhos = list(range(1, w.c_tot))
    o_by_step, g_gk = tiny.galois_keys([r * w.tokens for r in rhos])
    o_gks = {r: o_by_step[r * w.tokens] for r in rhos}
    want = tiny.o.ternary_matmul(o_cts, w.tokens, w.d_in, W, placement, o_gks)
    for mode in (1, 2):  # plain-ALU kernel, then the matrix-core kernel
        tiny.ctx.set_accumulate_mode(mode)
        out = tiny.ctx.ternary_matmul(g_gk, g_ct, w.tokens, w.d_in, W, placement)
        assert np.array_equal(out.export(), stack_cts(want)), "accumulate mode %d" % mode
        if mode == 1:
            out.free()
    tiny.ctx.set_accumulate_mode(0)
    assert out.limbs == tiny.pr.L and out.scale == g_ct.scale  # PCMM consumes no level
    ref = X @ W.astype(np.float64)
    err = 0.0
    dec = tiny.ctx.decrypt(tiny.g_sk, out)
    for i in range(w.d_out):
        p_i = 0 if placement == "zero" else i % w.c_tot
        err = max(err, np.abs(dec[i, p_i * w.tokens:(p_i + 1) * w.tokens] - ref[:, i]).max())
    assert err < 1e-3  # both placements (the oracle measures 3.6e-4 and 2.5e-4)
    out.free()
    g_ct.free()
    g_gk.free()


def test_matmul_paper_packing_needs_no_key(small4):
    """One column per ciphertext (c_tot = 1): the paper's own packing; pure add/sub."""
    p = small4
    d, m = 37, 70  # ragged against the 32-wide output tiles
    rng = np.random.default_rng(5)
    W = wl.ternary_weights(rng, d, m)
    W[:, 3] = 0  # an all-zero weight column gives the all-zero ciphertext
    X = rng.uniform(-1, 1, (p.n, d))
    for limbs in (p.pr.L, 3):
        o_cts, g_ct = p.encrypt_both(X.T, limbs)
        want = p.o.ternary_matmul(o_cts, p.n, d, W, "zero", {})
        for mode in (1, 2):
            p.ctx.set_accumulate_mode(mode)
            out = p.ctx.ternary_matmul(None, g_ct, p.n, d, W, "zero")
            got = out.export()
            assert np.array_equal(got, stack_cts(want)), "accumulate mode %d, limbs %d" % (mode, limbs)
            if mode == 1:
                out.free()
        p.ctx.set_accumulate_mode(0)
        assert not got[3].any()
        dec = p.ctx.decrypt(p.g_sk, out)
        assert np.abs(dec.T - X @ W.astype(np.float64)).max() < 1e-3
        out.free()
        g_ct.free()


def test_matmul_several_packed_inputs(small4):
    p = small4
    s, d, m = 64, 19, 13  # c_tot = 8: three packed inputs, the last one ragged
    rng = np.random.default_rng(6)
    W = wl.ternary_weights(rng, d, m)
    X = rng.uniform(-1, 1, (s, d))
    packed = wl.pack_columns(X, p.n)
    assert packed.shape[0] == 3
    o_cts, g_ct = p.encrypt_both(packed, p.pr.L)
    c_tot = p.n // s
    o_by_step, g_gk = p.galois_keys([r * s for r in range(1, c_tot)])
    o_gks = {r: o_by_step[r * s] for r in range(1, c_tot)}
    for placement in ("diagonal", "zero"):
        want = p.o.ternary_matmul(o_cts, s, d, W, placement, o_gks)
        for mode in (1, 2):
            p.ctx.set_accumulate_mode(mode)
            out = p.ctx.ternary_matmul(g_gk, g_ct, s, d, W, placement)
            assert np.array_equal(out.export(), stack_cts(want)), (placement, mode)
            if mode == 1:
                out.free()
        p.ctx.set_accumulate_mode(0)
        dec = p.ctx.decrypt(p.g_sk, out)
        ref = X @ W.astype(np.float64)
        for i in range(m):
            p_i = 0 if placement == "zero" else i % c_tot
            assert np.abs(dec[i, p_i * s:(p_i + 1) * s] - ref[:, i]).max() < 1e-3
        out.free()
    g_ct.free()
    g_gk.free()


def test_matmul_many_operands_and_wide_primes():
    """Long sums: 300 operands on 50-bit primes (matrix-core kernel, several k-steps, nine
    256-output tiles: one full group of eight plus a ragged one) and 40 operands on 60-bit primes (plain-ALU kernel with mid-loop reductions,
    the only valid one there)."""
    for params, d, m in (((8, 50, 3, 60, 1, 3, 40), 300, 2100), ((8, 60, 2, 61, 1, 2, 40), 40, 33)):
        p = Pair(params)
        try:
            rng = np.random.default_rng(8)
            W = wl.ternary_weights(rng, d, m)
            X = rng.uniform(-1, 1, (p.n, d)) * 0.05
            o_cts, g_ct = p.encrypt_both(X.T, p.pr.L)
            want = stack_cts(p.o.ternary_matmul(o_cts, p.n, d, W, "zero", {}))
            for mode in (1, 2):
                p.ctx.set_accumulate_mode(mode)
                out = p.ctx.ternary_matmul(None, g_ct, p.n, d, W, "zero")
                assert np.array_equal(out.export(), want), (params, mode)
                out.free()
            g_ct.free()
        finally:
            p.close()


@pytest.mark.parametrize("bits,operands,outputs,L", [
    (36, 513, 33, 3), (36, 768, 257, 3), (38, 769, 64, 3), (50, 512, 33, 3), (50, 513, 97, 3), (50, 1100, 257, 3), (54, 520, 40, 3),  # few words
    (36, 513, 513, 7), (36, 800, 600, 7), (50, 513, 769, 7), (50, 1100, 513, 7), (50, 700, 385, 8),  # shifted weights
    (36, 512, 513, 7), (50, 600, 384, 8), (50, 600, 512, 7), (50, 600, 600, 5), (38, 600, 600, 7)])  # one condition short of them
def test_signed_sums_by_digits(bits, operands, outputs, L):
    """Every way the words of the signed sums are cut into digits (7 bits with shifted weights: more than 512 operands and 384 outputs
    and at least 4096 pieces of 256 outputs x 32 words, below 2^36 and 2^50; 8 bits: the others) on the smallest and
    largest residues, ragged operand and output counts, and with the rescale between two layers applied on the way: plain
    integers, and the plain-ALU kernel on every word.  Only shifted weights need the sums of all operands."""
    import torch

    from paper_2509_09424_amd import binding
    ctx = binding.Context(12, bits, L, bits + 2, 1, 1, 20, seed=1)
    N, q = ctx.N, [int(x) for x in ctx.primes()[0]]
    W = np.random.default_rng(bits + operands).integers(-1, 2, (operands, outputs)).astype(np.int8)
    W[:, 0], W[:, 1] = 1, -1  # the largest sums of either sign
    x = torch.empty((operands, 2, L, N), dtype=torch.int64, device="cuda")
    for i in range(L):
        x[:, :, i].random_(0, q[i], generator=torch.Generator(device="cuda").manual_seed(i))
        x[:, :, i, :40] = q[i] - 1
    x[:, :, :, 40:80] = 0
    rows = [0, 1, outputs - 1]
    words = x[:, 1, :, 30:100].cpu().numpy().astype(object)
    want = np.stack([sum(int(W[v, r]) * words[v] for v in range(operands)) % np.array(q, dtype=object)[:, None] for r in rows])

    def product(mode, rescale):
        ctx.set_accumulate_mode(mode)
        limbs = L - rescale
        src, out = x.clone(), torch.full((outputs, 2, limbs, N), -1, dtype=torch.int64, device="cuda")
        h_in, h_out = ctx.ct_wrap(src.data_ptr(), operands, L, 1.0), ctx.ct_wrap(out.data_ptr(), outputs, limbs, 1.0)
        wt = ctx.weights_prepare(W, ctx.n_slots, operands, "zero", limbs)
        ctx.profile_enable(True)
        if rescale:
            ctx.rescale_ternary_matmul_prepared(h_in, 2.0 ** -5, wt, h_out)
        else:
            ctx.ternary_matmul_prepared(None, h_in, wt, h_out)
        torch.cuda.synchronize()
        items = 2 * limbs * (N // 32) * -(-outputs // 256)
        shifted = mode == 2 and operands > 512 and outputs > 384 and items >= 4096 and (bits <= 36 or 40 < bits <= 50)
        assert (ctx.profile_read().get("word_sums", (0, 0))[1] > 0) == shifted
        ctx.profile_enable(False)
        for h in (wt, h_in, h_out):
            h.free()
        return out

    try:
        for rescale in (False, True):
            plain, matrix = product(1, rescale), product(2, rescale)
            assert torch.equal(plain, matrix), "rescale %s" % rescale
            if not rescale:
                assert np.array_equal(matrix[rows, 1, :, 30:100].cpu().numpy().astype(object), want)
    finally:
        ctx.close()


@pytest.mark.parametrize("bits,operands,outputs", [
    (50, 1, 1), (36, 31, 32), (50, 33, 33), (38, 128, 129), (54, 129, 40), (50, 256, 300),  # all operands in LDS
    (50, 257, 128), (36, 300, 33), (38, 511, 129), (54, 257, 256), (50, 1025, 257), (54, 512, 384), (50, 2049, 8),  # in chunks
    (50, 384, 385), (36, 384, 520), (50, 385, 385), (54, 400, 600)])  # many outputs, and one condition past it
def test_signed_sums_of_few_operands_or_outputs(bits, operands, outputs):
    """Up to 384 operands or outputs the digits are formed where they are multiplied (with the rescale: up to 128 operands); largest and
    smallest residues among them, and one operand with weight +1 and one with -1 everywhere.  The plain-ALU kernel on every word, and plain
    integers."""
    import torch

    from paper_2509_09424_amd import binding
    L = 3
    ctx = binding.Context(12, bits, L, bits + 2, 1, 1, 20, seed=1)
    N, q = ctx.N, [int(x) for x in ctx.primes()[0]]
    W = np.random.default_rng(bits + operands).integers(-1, 2, (operands, outputs)).astype(np.int8)
    W[0], W[-1] = -1, 1
    W[:, 0] = 1
    x = torch.empty((operands, 2, L, N), dtype=torch.int64, device="cuda")
    for i in range(L):
        x[:, :, i].random_(0, q[i], generator=torch.Generator(device="cuda").manual_seed(i))
        x[:, :, i, :40] = q[i] - 1
    x[:, :, :, 40:80] = 0
    words = x[:, 1, :, 30:100].cpu().numpy().astype(object)
    want = sum(int(W[v, 0]) * words[v] for v in range(operands)) % np.array(q, dtype=object)[:, None]

    def product(mode, rescale):
        ctx.set_accumulate_mode(mode)
        limbs = L - rescale
        src, out = x.clone(), torch.full((outputs, 2, limbs, N), -1, dtype=torch.int64, device="cuda")
        h_in, h_out = ctx.ct_wrap(src.data_ptr(), operands, L, 1.0), ctx.ct_wrap(out.data_ptr(), outputs, limbs, 1.0)
        wt = ctx.weights_prepare(W, ctx.n_slots, operands, "zero", limbs)
        ctx.profile_enable(True)
        if rescale:
            ctx.rescale_ternary_matmul_prepared(h_in, 2.0 ** -5, wt, h_out)
        else:
            ctx.ternary_matmul_prepared(None, h_in, wt, h_out)
        torch.cuda.synchronize()
        ran = {k for k, v in ctx.profile_read().items() if v[1]}
        if mode == 2 and not (rescale and bits > 50):  # (wider primes: the rescale is a step of its own)
            few = operands <= 128 if rescale else operands <= 384 or outputs <= 384
            assert ("rescale_accumulate_direct" if rescale else "accumulate_direct") in ran if few else "accumulate_mfma" in ran, ran
        ctx.profile_enable(False)
        for h in (wt, h_in, h_out):
            h.free()
        return out

    try:
        for rescale in (False, True):
            plain, matrix = product(1, rescale), product(2, rescale)
            assert torch.equal(plain, matrix), "rescale %s" % rescale
            if not rescale:
                assert np.array_equal(matrix[0, 1, :, 30:100].cpu().numpy().astype(object), want)
    finally:
        ctx.close()


@pytest.mark.parametrize("log_n,bits,operands,outputs,rescale,kernel", [
    (10, 50, 256, 384, 0, "accumulate_direct"), (10, 50, 256, 385, 0, "accumulate_mfma"), (10, 36, 16, 960, 0, "accumulate_direct"), (10, 36, 16, 961, 0, "accumulate_mfma"),
    (10, 54, 300, 600, 0, "accumulate_mfma"), (10, 50, 769, 40, 0, "accumulate_mfma"),
    (16, 50, 128, 129, 1, "rescale_accumulate_direct"), (16, 36, 31, 600, 1, "rescale_accumulate_direct"), (16, 50, 129, 40, 1, "accumulate_mfma"),
    (16, 50, 384, 390, 0, "accumulate_direct"), (16, 36, 300, 33, 0, "accumulate_direct")])
def test_signed_sums_on_the_smallest_and_largest_rings(log_n, bits, operands, outputs, rescale, kernel):
    """Two limbs: fewer word tiles than compute units, on both sides of the lines, and many, also with the rescale.  The plain-ALU kernel on every word."""
    import torch

    from paper_2509_09424_amd import binding
    L = 2 + rescale
    ctx = binding.Context(log_n, bits, L, bits + 2, 1, 1, 20, seed=1)
    q = [int(x) for x in ctx.primes()[0]]
    W = np.random.default_rng(operands).integers(-1, 2, (operands, outputs)).astype(np.int8)
    x = torch.empty((operands, 2, L, ctx.N), dtype=torch.int64, device="cuda")
    for i in range(L):
        x[:, :, i].random_(0, q[i], generator=torch.Generator(device="cuda").manual_seed(i))
    got = []
    for mode in (1, 2):
        ctx.set_accumulate_mode(mode)
        out = torch.full((outputs, 2, 2, ctx.N), -1, dtype=torch.int64, device="cuda")
        src = x.clone()
        h_in, h_out = ctx.ct_wrap(src.data_ptr(), operands, L, 1.0), ctx.ct_wrap(out.data_ptr(), outputs, 2, 1.0)
        wt = ctx.weights_prepare(W, ctx.n_slots, operands, "zero", 2)
        ctx.profile_enable(True)
        if rescale:
            ctx.rescale_ternary_matmul_prepared(h_in, 2.0 ** -5, wt, h_out)
        else:
            ctx.ternary_matmul_prepared(None, h_in, wt, h_out)
        torch.cuda.synchronize()
        ran = {k for k, v in ctx.profile_read().items() if v[1]}
        assert mode == 1 or kernel in ran, ran
        ctx.profile_enable(False)
        got.append(out)
        for h in (wt, h_in, h_out):
            h.free()
    assert torch.equal(*got)
    ctx.close()


@pytest.mark.parametrize("bits,operands,kernel", [(50, 8192, "accumulate_mfma"), (50, 8193, "accumulate"), (36, 32768, "accumulate_mfma"),
                                                  (36, 32769, "accumulate")])
def test_signed_sums_at_the_most_operands(bits, operands, kernel):
    """The most operands that the matrix cores are given: at 50 bits the sum of all operands of a word comes just under 2^63, at 36
    bits a sum of one digit reaches 2^23.  Largest residues throughout, with a row of weights +1 and one of -1, so that every
    bound of the recombination is met; one operand more goes to the plain-ALU kernel.  Plain integers."""
    import torch

    from paper_2509_09424_amd import binding
    L, outputs = 6, 513
    ctx = binding.Context(12, bits, L, bits + 2, 1, 1, 20, seed=1)
    try:
        N, q = ctx.N, [int(x) for x in ctx.primes()[0]]
        W = np.random.default_rng(operands).integers(-1, 2, (operands, outputs)).astype(np.int8)
        W[:, 0], W[:, 1], W[:, 2] = 1, -1, 0
        x = torch.empty((operands, 2, L, N), dtype=torch.int64, device="cuda")
        for i in range(L):
            x[:, :, i] = q[i] - 1
            x[:, :, i, 1::4] = 0
            x[:, :, i, 2::4].random_(0, q[i], generator=torch.Generator(device="cuda").manual_seed(i))
            x[:, :, i, 3::4] = (q[i] - 1) // 2
        out = torch.full((outputs, 2, L, N), -1, dtype=torch.int64, device="cuda")
        h_in, h_out = ctx.ct_wrap(x.data_ptr(), operands, L, 1.0), ctx.ct_wrap(out.data_ptr(), outputs, L, 1.0)
        wt = ctx.weights_prepare(W, ctx.n_slots, operands, "zero", L)
        ctx.profile_enable(True)
        ctx.ternary_matmul_prepared(None, h_in, wt, h_out)
        torch.cuda.synchronize()
        ran = {k for k, v in ctx.profile_read().items() if v[1]}
        assert kernel in ran and ("word_sums" in ran) == (kernel == "accumulate_mfma"), ran
        # every word: three of four are the same for all operands; the others are taken as halves of 25 bits, whose sums a
        # product of doubles has exactly
        total = torch.from_numpy(W.sum(0, dtype=np.int64)).cuda()
        Wd = torch.from_numpy(W).cuda().double()
        for i in range(L):
            for k, value in ((0, q[i] - 1), (1, 0), (3, (q[i] - 1) // 2)):
                want = torch.tensor([int(t) * value % q[i] for t in total.tolist()], device="cuda")
                assert torch.equal(out[:, :, i, k::4], want[:, None, None].expand(outputs, 2, N // 4)), (i, k)
            r = x[:, :, i, 2::4].reshape(operands, -1)
            low, high = (Wd.T @ (r & 0x1ffffff).double()).long(), (Wd.T @ (r >> 25).double()).long()
            want = high % q[i]
            for _ in range(5):  # times 2^25
                want = want * 32 % q[i]
            want = (want + low) % q[i]
            assert torch.equal(out[:, :, i, 2::4].reshape(outputs, -1), want), i
        for h in (wt, h_in, h_out):
            h.free()
    finally:
        ctx.close()


def test_mul_scalar_rescale_bit_exact_and_two_layer(small4):
    p = small4
    rng = np.random.default_rng(7)
    z = rng.uniform(-1, 1, (2, p.n))
    for kappa in (2.0 ** -5, -0.3):
        o_cts, g_ct = p.encrypt_both(z, p.pr.L)
        want = [p.o.mul_scalar_rescale(c, kappa) for c in o_cts]
        p.ctx.mul_scalar_rescale(g_ct, kappa)
        assert g_ct.limbs == p.pr.L - 1
        assert np.array_equal(g_ct.export(), stack_cts(want))
        assert g_ct.scale == want[0].scale
        dec = p.ctx.decrypt(p.g_sk, g_ct)
        assert np.abs(dec - kappa * z).max() < 1e-3
        # a rotation after the rescale runs at the lower level on the strided storage
        o_gks, g_gk = p.galois_keys([2])
        rot = p.ctx.rotate(g_gk, g_ct, [2, 2])
        want_rot = [p.o.rotate(c, o_gks[2]) for c in want]
        assert np.array_equal(rot.export(), stack_cts(want_rot))
        rot.free()
        g_gk.free()
        g_ct.free()


def test_rescale_fused_into_second_layer_bit_exact(small4):
    """Scalar-multiply + rescale applied while the second layer's accumulate reads its operands
    (one call) against the oracle's two steps, on both accumulate paths and for a ragged operand count."""
    p = small4
    d, m = 37, 70
    rng = np.random.default_rng(9)
    W = wl.ternary_weights(rng, d, m)
    X = rng.uniform(-1, 1, (p.n, d))
    for limbs, kappa in ((p.pr.L, 2.0 ** -5), (3, -0.3)):
        o_cts, _ = p.encrypt_both(X.T, limbs)
        o_mid = [p.o.mul_scalar_rescale(c, kappa) for c in o_cts]
        want = stack_cts(p.o.ternary_matmul(o_mid, p.n, d, W, "zero", {}))
        for mode in (1, 2):
            g_ct = p.ctx.ct_import(stack_cts(o_cts), o_cts[0].scale)
            p.ctx.set_accumulate_mode(mode)
            out = p.ctx.rescale_ternary_matmul(g_ct, kappa, W)
            assert out.limbs == limbs - 1 and g_ct.limbs == limbs - 1
            assert np.array_equal(out.export(), want), "accumulate mode %d, limbs %d" % (mode, limbs)
            assert out.scale == o_mid[0].scale == g_ct.scale
            if mode == 2:
                dec = p.ctx.decrypt(p.g_sk, out)
                assert np.abs(dec.T - (kappa * X) @ W.astype(np.float64)).max() < 1e-3
            out.free()
            g_ct.free()
        p.ctx.set_accumulate_mode(0)
    E = p.binding.EnsiError
    one = p.ctx.ct_import(stack_cts(o_cts)[:, :, :1], 1.0)
    dst = p.ctx.ct_alloc(m, 1)
    with pytest.raises(E, match="code -3"):
        p.ctx.rescale_ternary_matmul(one, 0.5, W, dst)  # no limb left to drop
    dst.free()
    one.free()


def test_error_paths(tiny):
    E = tiny.binding.EnsiError
    z = np.zeros((1, tiny.n))
    _, g_ct = tiny.encrypt_both(z, tiny.pr.L)
    _, g_gk = tiny.galois_keys([1])
    with pytest.raises(E, match="code -2"):
        tiny.ctx.rotate(g_gk, g_ct, [2])  # no key for step 2
    W = np.zeros((64, 64), dtype=np.int8)
    W[0, 0] = 2
    with pytest.raises(E, match="code -1"):
        tiny.ctx.ternary_matmul(g_gk, g_ct, 32, 64, W)
    W[0, 0] = 1
    W[5, 0] = 1
    with pytest.raises(E, match="code -2"):
        tiny.ctx.ternary_matmul(None, g_ct, 32, 64, W, "zero")  # needs rotations, no key set
    with pytest.raises(E, match="code -4"):
        tiny.ctx.ternary_matmul(g_gk, g_ct, 32, 4000, np.zeros((4000, 2), dtype=np.int8))  # needs 2 packed inputs
    low = tiny.ctx.ct_alloc(1, 2)
    with pytest.raises(E, match="code -3"):
        tiny.ctx.rotate(g_gk, g_ct, [1], low)
    low.free()
    g_ct.free()
    g_gk.free()


# ---------------------------------------------------------------- full ring (N = 2^16)
KEYSWITCH = wl.WORKLOADS[1].param_tuple()  # 10 x 50-bit + 3 x 60-bit, alpha = 3


@pytest.fixture(scope="module")
def full():
    p = Pair(KEYSWITCH)
    yield p
    p.close()


def test_full_ring_ntt_roundtrip_and_evaluation_set(full):
    """The N = 2^16 transform (register radix-16 steps; fp64 arithmetic on the 50-bit primes,
    signed multiply-adds on the 60-bit ones)."""
    rng = np.random.default_rng(10)
    L = full.pr.L
    primes = full.pr.q + full.pr.p
    idx = [0, L - 1, L, L + 2]  # two 50-bit primes, two 60-bit primes
    x = np.stack([rng.integers(0, full.pr.q[-1], size=full.N, dtype=np.uint64) for _ in idx])
    x[0, :4] = [0, 1, full.pr.q[0] - 1, full.pr.q[0] // 2]
    x[0] %= np.uint64(full.pr.q[0])
    ct = full.ctx.ct_import(x.reshape(2, 2, 1, full.N) % np.uint64(full.pr.q[0]), 1.0)
    x = ct.export().reshape(4, full.N)
    full.ctx.ntt(ct.device_ptr, idx, inverse=False)
    fwd = ct.export().reshape(4, full.N)
    want = full.o.ntt(x, [primes[i] for i in idx])
    assert np.array_equal(np.sort(fwd, axis=1), np.sort(want, axis=1))
    full.ctx.ntt(ct.device_ptr, idx, inverse=True)
    assert np.array_equal(ct.export().reshape(4, full.N), x)
    ct.free()


@pytest.mark.parametrize("params", [(16, 60, 28, 61, 4, 4, 40), (12, 60, 6, 60, 2, 2, 40)], ids=["64K", "4K"])
def test_ntt_of_ciphertext_primes_below_2_60(params):
    """Primes from next to 2^60 down to the far end of the range of the signed arithmetic for them (the 28th of the
    2^16 ring is 0.79 2^26 below), at extreme residues: all q - 1, all (q - 1) / 2, alternating, random."""
    import torch
    from paper_2509_09424_amd import binding
    from oracle import Oracle, Params
    ctx, o = binding.Context(*params, seed=1), Oracle(Params(*params))
    N, primes = ctx.N, [q for q in ctx.primes()[0]]
    rng = np.random.default_rng(14)
    rows, idx = [], []
    for i in sorted({0, len(primes) // 2, len(primes) - 1}):
        q = np.uint64(primes[i])
        alternating = np.zeros(N, dtype=np.uint64)
        alternating[::2] = q - np.uint64(1)
        rows += [np.full(N, q - np.uint64(1)), np.full(N, (q - np.uint64(1)) // np.uint64(2)), alternating, rng.integers(0, q, size=N, dtype=np.uint64)]
        idx += [i] * 4
    x = np.stack(rows)
    for inverse in (False, True):
        buf = torch.from_numpy(x.view(np.int64)).cuda()
        for r in range(0, len(idx), 4):  # (the primes of a call repeat with a period: one call per prime)
            ctx.ntt(buf[r].data_ptr(), idx[r:r + 4], inverse=inverse)
        torch.cuda.synchronize()
        got = buf.cpu().numpy().view(np.uint64)
        if not inverse:
            want = o.ntt(x, [primes[i] for i in idx])
            assert np.array_equal(np.sort(got, axis=1), np.sort(want, axis=1))
        for r in range(0, len(idx), 4):
            ctx.ntt(buf[r].data_ptr(), idx[r:r + 4], inverse=not inverse)
        torch.cuda.synchronize()
        assert np.array_equal(buf.cpu().numpy().view(np.uint64), x), inverse
    ctx.close()


def test_full_ring_ntt_batch_with_ragged_groups(full):
    """A batch whose limbs cycle through three primes (two below 2^50, one above) and whose count leaves the last
    group of every prime incomplete: the row pass runs a tile for up to eight limbs of one prime per block."""
    import torch
    rng = np.random.default_rng(12)
    L = full.pr.L
    primes = full.pr.q + full.pr.p
    pattern = [1, L + 1, L - 1]
    n = 29  # 10, 10 and 9 limbs per prime: groups of 8 + 2, 8 + 2, 8 + 1
    idx = [pattern[r % 3] for r in range(n)]
    x = np.stack([rng.integers(0, primes[i], size=full.N, dtype=np.uint64) for i in idx])
    buf = torch.from_numpy(x.view(np.int64)).cuda()
    full.ctx.ntt(buf.data_ptr(), idx, inverse=False)
    torch.cuda.synchronize()
    fwd = buf.cpu().numpy().view(np.uint64)
    for r in (0, 1, 2, 23, 24, 26, 27, 28):  # first limbs, and the limbs of the incomplete groups
        want = full.o.ntt(x[r:r + 1], [primes[idx[r]]])[0]
        assert np.array_equal(np.sort(fwd[r]), np.sort(want)), r
    # limbs of one prime are transformed alike: same input -> same output, whatever its place in a group
    y = x.copy()
    y[27] = x[0]
    buf2 = torch.from_numpy(y.view(np.int64)).cuda()
    full.ctx.ntt(buf2.data_ptr(), idx, inverse=False)
    torch.cuda.synchronize()
    assert np.array_equal(buf2[27].cpu().numpy(), buf[0].cpu().numpy())
    full.ctx.ntt(buf.data_ptr(), idx, inverse=True)
    torch.cuda.synchronize()
    assert np.array_equal(buf.cpu().numpy().view(np.uint64), x)


def test_full_ring_rotate_bit_exact(full):
    p = full
    steps = [1, -1, 4096]
    o_gks, g_gk = p.galois_keys(sorted(set(steps)))
    z = p.rng.uniform(-1, 1, (len(steps), p.n))
    for limbs in (p.pr.L, 4):
        o_cts, g_ct = p.encrypt_both(z, limbs)
        assert np.array_equal(g_ct.export(), stack_cts(o_cts))
        out = p.ctx.rotate(g_gk, g_ct, steps)
        want = [p.o.rotate(c, o_gks[st]) for c, st in zip(o_cts, steps)]
        assert np.array_equal(out.export(), stack_cts(want)), "limbs=%d" % limbs
        dec = p.ctx.decrypt(p.g_sk, out, 0, 256)
        for i, st in enumerate(steps):
            assert np.abs(dec[i] - np.roll(z[i], -st)[:256]).max() < 1e-3
        out.free()
        g_ct.free()
    g_gk.free()


def test_full_ring_rotate_all_sixteen_galois_elements(full, capsys):
    """The key-switch microbenchmark's own step set at the full level: one ciphertext per Galois element (steps
    2^0 .. 2^14 and -1), every one bit-exact against the oracle and a left shift of the slots after decryption."""
    p = full
    steps = list(wl.KEYSWITCH_STEPS)
    assert len(steps) == 16 and len({p.pr.galois_element(st) for st in steps}) == 16
    o_gks, g_gk = p.galois_keys(steps)
    z = p.rng.uniform(-1, 1, (len(steps), p.n))
    o_cts, g_ct = p.encrypt_both(z, p.pr.L)
    out = p.ctx.rotate(g_gk, g_ct, steps)
    got = out.export()
    for i, st in enumerate(steps):
        assert np.array_equal(got[i], p.o.rotate(o_cts[i], o_gks[st]).limbs()), "step %d" % st
    dec = p.ctx.decrypt(p.g_sk, out)
    err = max(np.abs(dec[i] - np.roll(z[i], -st)).max() for i, st in enumerate(steps))
    assert err < 1e-3
    with capsys.disabled():
        print("\n[cfg 2, alpha = 3] 16 Galois elements bit-exact; decrypted max abs error %.3e" % err, flush=True)
    out.free()
    g_ct.free()
    g_gk.free()


def test_full_ring_rotate_literal_three_digits(capsys):
    """The literal reading of "dnum = 3" for the key-switch configuration: 10 ciphertext primes in three digits of
    4, 4 and 2 limbs (alpha = 4) against three special primes.  A digit is then larger than P, so the switching
    noise is far above the 1e-3 bound: parity (which does not depend on the noise) is gated, the decrypted error is
    only reported."""
    w = wl.WORKLOADS[1]
    p = Pair((w.log_n, w.q_bits, w.q_count, w.p_bits, w.p_count, 4, w.log_scale))
    try:
        assert p.pr.beta(p.pr.L) == 3
        steps = [1, -1, 1 << 7, 1 << 14]
        o_gks, g_gk = p.galois_keys(steps)
        z = p.rng.uniform(-1, 1, (len(steps), p.n))
        o_cts, g_ct = p.encrypt_both(z, p.pr.L)
        out = p.ctx.rotate(g_gk, g_ct, steps)
        got = out.export()
        for i, st in enumerate(steps):
            assert np.array_equal(got[i], p.o.rotate(o_cts[i], o_gks[st]).limbs()), "step %d" % st
        dec = p.ctx.decrypt(p.g_sk, out)
        err = max(np.abs(dec[i] - np.roll(z[i], -st)).max() for i, st in enumerate(steps))
        with capsys.disabled():
            print("\n[cfg 2, literal alpha = 4, beta = 3] bit-exact; decrypted max abs error %.3e (reported, not gated)" % err, flush=True)
        out.free()
        g_ct.free()
        g_gk.free()
    finally:
        p.close()


def test_full_ring_matmul_bit_exact(full):
    p = full
    s, d, m = p.n // 4, 6, 5  # c_tot = 4: two packed inputs, rotations by 1..3 blocks
    rng = np.random.default_rng(11)
    W = wl.ternary_weights(rng, d, m)
    W[0, 0], W[5, 4] = 1, -1
    X = np.clip(rng.standard_normal((s, d)), -4, 4)
    packed = wl.pack_columns(X, p.n)
    o_cts, g_ct = p.encrypt_both(packed, p.pr.L)
    o_by_step, g_gk = p.galois_keys([r * s for r in range(1, 4)])
    o_gks = {r: o_by_step[r * s] for r in range(1, 4)}
    want = stack_cts(p.o.ternary_matmul(o_cts, s, d, W, "diagonal", o_gks))
    for mode in (1, 2):
        p.ctx.set_accumulate_mode(mode)
        out = p.ctx.ternary_matmul(g_gk, g_ct, s, d, W, "diagonal")
        assert np.array_equal(out.export(), want), "accumulate mode %d" % mode
        if mode == 1:
            out.free()
    p.ctx.set_accumulate_mode(0)
    ref = X @ W.astype(np.float64)
    for i in range(m):
        one = p.ctx.decrypt(p.g_sk, out, (i % 4) * s, 512)
        assert np.abs(one[i] - ref[:512, i]).max() < 1e-3
    out.free()
    g_ct.free()
    g_gk.free()


@pytest.mark.parametrize("params,why", [
    ((16, 45, 4, 48, 2, 2, 36), "every prime below 2^50: the special limbs take the fp64 path of the fused kernels too"),
    ((16, 55, 3, 60, 1, 2, 40), "ciphertext primes above 2^50: the unfused integer kernels at N = 2^16"),
], ids=["all-fp", "wide-q"])
def test_full_ring_rotate_other_prime_sizes(params, why):
    p = Pair(params)
    steps = [3, -5]
    o_gks, g_gk = p.galois_keys(steps)
    z = p.rng.uniform(-1, 1, (len(steps), p.n))
    for limbs in (p.pr.L, 1):
        o_cts, g_ct = p.encrypt_both(z, limbs)
        out = p.ctx.rotate(g_gk, g_ct, steps)
        want = [p.o.rotate(c, o_gks[st]) for c, st in zip(o_cts, steps)]
        assert np.array_equal(out.export(), stack_cts(want)), (why, limbs)
        out.free()
        g_ct.free()
    g_gk.free()
    p.close()


@pytest.mark.parametrize("params", [(12, 50, 5, 60, 4, 4, 40), (14, 50, 6, 60, 2, 2, 40)], ids=["4K", "16K"])
def test_few_and_many_rotations_of_a_raised_input_bit_exact(params):
    """Around the two rotations per raised ciphertext up to which the inner product runs the digits' row passes itself: one to
    three on one input, and on two inputs four (still two each) and five."""
    p = Pair(params)
    s = p.n // 4
    o_gks, g_gk = p.galois_keys([s, 2 * s, 3 * s])
    rng = np.random.default_rng(8)
    for d in (2, 3, 4, 6, 7):
        W = wl.ternary_weights(rng, d, 3)
        o_cts, g_ct = p.encrypt_both(wl.pack_columns(rng.uniform(-1, 1, (s, d)), p.n), p.pr.L)
        out = p.ctx.ternary_matmul(g_gk, g_ct, s, d, W, "zero")
        want = p.o.ternary_matmul(o_cts, s, d, W, "zero", {r: o_gks[r * s] for r in range(1, 4)})
        assert np.array_equal(out.export(), stack_cts(want)), d
        out.free()
        g_ct.free()
    g_gk.free()
    p.close()


@pytest.mark.parametrize("params", [
    (12, 50, 5, 60, 4, 4, 40), (13, 50, 5, 60, 3, 2, 40), (14, 50, 6, 60, 2, 2, 40), (15, 50, 4, 60, 1, 1, 36),  # special primes just below 2^60
    (12, 45, 4, 48, 3, 3, 36),  # every prime in fp64
    (13, 50, 3, 61, 2, 2, 40), (12, 50, 3, 55, 4, 1, 36),  # special primes in neither of the two fast arithmetics
], ids=["4K-wide4", "8K-wide3", "16K-wide2", "32K-wide1", "4K-fp3", "8K-61bit", "4K-55bit"])
def test_register_transform_rings_bit_exact(params):
    """Every ring of the register transform and every kind and number of special primes: rotations that have their raised
    ciphertext to themselves, and rotations (of a product) that share one."""
    p = Pair(params)
    s = p.n // 4
    steps = [s, 2 * s, 3 * s, -1]
    o_gks, g_gk = p.galois_keys(steps)
    z = p.rng.uniform(-1, 1, (3, p.n))
    for limbs in (p.pr.L, 2):
        o_cts, g_ct = p.encrypt_both(z, limbs)
        assert np.array_equal(g_ct.export(), stack_cts(o_cts))
        dec = p.ctx.decrypt(p.g_sk, g_ct)
        assert np.abs(dec - z).max() < 1e-3
        part = p.ctx.decrypt(p.g_sk, g_ct, p.n // 3, 11)  # a window of slots; the values are exact sums in double precision
        assert np.abs(part - dec[:, p.n // 3:p.n // 3 + 11]).max() <= 1e-13 * np.abs(dec).max()
        for n in (1, 3):
            one = p.ctx.ct_import(stack_cts(o_cts[:n]), g_ct.scale)
            out = p.ctx.rotate(g_gk, one, [-1, s, s][:n])
            want = [p.o.rotate(c, o_gks[st]) for c, st in zip(o_cts, [-1, s, s][:n])]
            assert np.array_equal(out.export(), stack_cts(want)), (limbs, n)
            out.free()
            one.free()
        g_ct.free()
    # encode: slots that do not fill the ring
    pt = p.ctx.encode(z[:, :p.n - 3], p.pr.L)
    want = np.stack([p.o.encode_coeffs(np.concatenate([v[:p.n - 3], np.zeros(3)])) for v in z])
    got = p.ctx.pt_export(pt)
    assert np.abs(got - want).max() <= 1 and (got != want).mean() < 0.01
    pt.free()
    one = p.ctx.encrypt(p.g_pk, p.ctx.pt_import(want, 1))  # a single limb: decrypted without the combination of two
    assert np.abs(p.ctx.decrypt(p.g_sk, one)[:, :p.n - 3] - z[:, :p.n - 3]).max() < 1e-3
    one.free()
    rng = np.random.default_rng(3)
    d, m = 6, 5
    W = wl.ternary_weights(rng, d, m)
    o_cts, g_ct = p.encrypt_both(wl.pack_columns(rng.uniform(-1, 1, (s, d)), p.n), p.pr.L)
    out = p.ctx.ternary_matmul(g_gk, g_ct, s, d, W, "diagonal")
    want = p.o.ternary_matmul(o_cts, s, d, W, "diagonal", {r: o_gks[r * s] for r in range(1, 4)})
    assert np.array_equal(out.export(), stack_cts(want))
    out.free()
    g_ct.free()
    g_gk.free()
    p.close()


@pytest.mark.parametrize("params", [(12, 50, 8, 60, 1, 1, 40), (12, 50, 7, 60, 2, 1, 40), (13, 45, 8, 48, 1, 1, 36), (12, 50, 8, 61, 1, 1, 40)],
                         ids=["4K-wide-8", "4K-wide-7", "8K-fp-8", "4K-61bit-8"])
def test_inner_products_of_one_to_eight_digits(params):
    """Sums of up to eight products that are reduced once, over digits that several rotations share: every number of digits, for every kind of
    special primes, and numbers of rotations around the four of a block; then groups of rotations (a fill)."""
    p = Pair(params)
    s = p.n // 8
    fill = p.ctx.fill_steps(1, p.n)
    o_gks, g_gk = p.galois_keys(sorted({r * s for r in range(1, 8)} | set(fill)))
    rng = np.random.default_rng(12)
    for limbs in range(p.pr.L, 0, -1):
        d = 8 - limbs % 5
        W = np.ones((d, 1), dtype=np.int8)
        o_cts, g_ct = p.encrypt_both(wl.pack_columns(rng.uniform(-1, 1, (s, d)), p.n), limbs)
        out = p.ctx.ternary_matmul(g_gk, g_ct, s, d, W, "zero")
        want = p.o.ternary_matmul(o_cts, s, d, W, "zero", {r: o_gks[r * s] for r in range(1, d)})
        assert np.array_equal(out.export(), stack_cts(want)), (limbs, d)
        out.free()
        g_ct.free()
    o_cts, g_ct = p.encrypt_both(p.rng.uniform(-1, 1, (1, p.n)), p.pr.L)
    masks = p.o.one_hot_masks([5], p.pr.L)
    g_masks = p.ctx.pt_set_scale(p.ctx.pt_import(masks, p.pr.L), float(p.pr.q[-1]))
    out = p.ctx.replicate(g_gk, g_ct, [0], g_masks, [0])
    assert np.array_equal(out.export(), stack_cts([p.o.replicate(o_cts[0], masks[0], {st: o_gks[st] for st in fill})]))
    for h in (g_ct, g_masks, out, g_gk):
        h.free()
    p.close()


@pytest.mark.parametrize("params", [(12, 50, 5, 60, 3, 2, 40), (12, 45, 4, 48, 2, 2, 36), (13, 50, 3, 61, 2, 1, 40), (12, 50, 8, 60, 1, 1, 40), (12, 50, 4, 55, 4, 1, 36)],
                         ids=["4K-wide3", "4K-fp2", "8K-61bit2", "4K-eight-digits", "4K-55bit4"])
def test_rotations_of_few_and_more_ciphertexts(params):
    """The forms of the key switch that few rotations take (a limb to a block, special limbs first, a wave to each digit) and the
    ones beyond, around the batch sizes where they change, for every kind and number of special primes."""
    p = Pair(params)
    steps = [1, -1, p.n // 2]
    o_gks, g_gk = p.galois_keys(steps)
    o_cts, g_ct = p.encrypt_both(p.rng.uniform(-1, 1, (2, p.n)), p.pr.L)
    both = stack_cts(o_cts)
    want = np.stack([stack_cts([p.o.rotate(c, o_gks[st]) for c in o_cts]) for st in steps])
    for n in (1, 2, 9, 16, 17, 33, 47, 64, 65, 128, 129):
        which, st = np.arange(n) % 2, np.arange(n) // 2 % 3
        batch = p.ctx.ct_import(np.ascontiguousarray(both[which]), g_ct.scale)
        out = p.ctx.rotate(g_gk, batch, [steps[k] for k in st])
        assert np.array_equal(out.export(), want[st, which]), n
        out.free()
        batch.free()
    for h in (g_ct, g_gk):
        h.free()
    p.close()


@pytest.mark.parametrize("params", [(14, 50, 6, 60, 2, 2, 40), (14, 45, 4, 48, 2, 1, 36), (15, 50, 4, 61, 2, 2, 40), (15, 50, 3, 60, 1, 1, 40), (16, 50, 5, 60, 3, 2, 40),
                                    (16, 45, 4, 48, 2, 1, 36), (16, 50, 3, 61, 2, 1, 40)], ids=["16K", "16K-fp", "32K-61bit", "32K", "64K", "64K-fp", "64K-61bit"])
def test_few_rotations_on_large_rings(params):
    """The same forms on the rings from 2^14: up to 512 waves of four rows a digit to a wave, then two and three ciphertexts past them."""
    p = Pair(params)
    steps = [1, -1]
    o_gks, g_gk = p.galois_keys(steps)
    o_cts, g_ct = p.encrypt_both(p.rng.uniform(-1, 1, (2, p.n)), p.pr.L)
    both = stack_cts(o_cts)
    want = np.stack([stack_cts([p.o.rotate(c, o_gks[st]) for c in o_cts]) for st in steps])
    for n in (1, 2, 3, 9):
        which, st = np.arange(n) % 2, np.arange(n) // 2 % 2
        batch = p.ctx.ct_import(np.ascontiguousarray(both[which]), g_ct.scale)
        out = p.ctx.rotate(g_gk, batch, [steps[k] for k in st])
        assert np.array_equal(out.export(), want[st, which]), n
        out.free()
        batch.free()
    for h in (g_ct, g_gk):
        h.free()
    p.close()


@pytest.mark.parametrize("log_n,n", [(12, 300), (13, 5), (14, 70), (15, 3), (16, 37)])
def test_client_transforms_equal_the_length_2n_transform(log_n, n):
    """Encoding and decoding by the kernels of the register transform against the length-2N transform, which a context with
    55-bit ciphertext primes runs: the same coefficients and the same slots to the last bit (neither depends on the
    primes), at batches of several chunks with a ragged last one, and at scales where a coefficient hangs on the last bit."""
    from paper_2509_09424_amd import binding
    ctx = {bits: binding.Context(log_n, bits, 2, 60, 1, 1, 43, seed=1) for bits in (50, 55)}
    N, rng = 1 << log_n, np.random.default_rng(log_n)
    z = rng.uniform(-1, 1, (n, N // 2 - 3))
    for slots, scale in ((z, None), (z[:2, :11], None), (z * 2.0 ** -8, 2.0 ** 55)):
        got = {}
        for bits, c in ctx.items():
            pt = c.encode(slots, 2) if scale is None else c.encode_at(slots, 2, scale)
            got[bits] = c.pt_export(pt)
            pt.free()
        assert np.array_equal(got[50], got[55]), scale
    # coefficients up to the end of the 64-bit range, beyond what a double or one prime holds: from their residues modulo two
    # primes (an encryption with no randomness is the plaintext itself)
    big = {}
    for bits, c in ctx.items():
        _, pk = c.keygen(None, None, 5)
        pt = c.encode_at(0.9 + 0.1 * z[:1], 2, 2.0 ** 62)
        none = np.zeros((1, N), dtype=np.int8)
        ct = c.encrypt(pk, pt, none, none, none)
        q, r = c.primes()[0], ct.export()[0, 0].astype(object)
        m = (r[0] + q[0] * ((r[1] - r[0]) * pow(q[0], -1, q[1]) % q[1])) % (q[0] * q[1])
        big[bits] = np.where(m > q[0] * q[1] // 2, m - q[0] * q[1], m)
        for h in (pt, ct, pk):
            h.free()
    assert max(abs(x) for x in big[50]) > 1 << 61 and np.array_equal(big[50], big[55])
    # decoding: ciphertexts that are plaintexts
    m = rng.integers(-2 ** 44, 2 ** 44, (min(n, 19 if log_n == 16 else n), N))
    for limbs in (1, 2):
        out = {}
        for bits, c in ctx.items():
            sk, pk = c.keygen(None, None, 5)
            words = np.zeros((len(m), 2, limbs, N), dtype=np.uint64)
            for i in range(limbs):
                words[:, 0, i] = m % c.primes()[0][i]
            ct = c.ct_import(words, 2.0 ** 43)
            out[bits] = c.decrypt(sk, ct), c.decrypt(sk, ct, N // 6, 17)
            for h in (ct, sk, pk):
                h.free()
        assert np.array_equal(out[50][0], out[55][0]) and np.array_equal(out[50][1], out[55][1]), limbs
        assert np.array_equal(out[50][1], out[50][0][:, N // 6:N // 6 + 17]), limbs
    for c in ctx.values():
        c.close()


@pytest.mark.parametrize("log_n,n", [(12, 259), (16, 19)])
def test_encrypt_and_decrypt_batches_of_several_chunks(log_n, n):
    """A batch longer than one chunk, the last chunk ragged, gives the words and the slots of its ciphertexts one part at a time."""
    from paper_2509_09424_amd import binding
    c = binding.Context(log_n, 50, 3, 60, 1, 1, 40, seed=1)
    rng = np.random.default_rng(9)
    sk, pk = c.keygen(None, None, 5)
    z = rng.uniform(-1, 1, (n, c.n_slots))
    small = [wl.ternary_poly(rng, (n, c.N)), wl.error_poly(rng, (n, c.N)), wl.error_poly(rng, (n, c.N))]
    pt = c.encode(z, 3)
    ct = c.encrypt(pk, pt, *small)
    words, slots = ct.export(), c.decrypt(sk, ct)
    assert np.abs(slots - z).max() < 1e-3
    for a, b in ((0, 1), (1, n // 2), (n // 2, n - 1), (n - 1, n)):
        part = c.encode(z[a:b], 3)
        part_ct = c.encrypt(pk, part, *[x[a:b] for x in small])
        assert np.array_equal(part_ct.export(), words[a:b]) and np.array_equal(c.decrypt(sk, part_ct), slots[a:b]), (a, b)
        for h in (part, part_ct):
            h.free()
    for h in (pt, ct, sk, pk):
        h.free()
    c.close()


def test_encode_after_an_allocation_that_failed(small4):
    """A batch larger than any card is refused, and the next calls work."""
    from paper_2509_09424_amd import binding
    ctx = binding.Context(12, 50, 4, 60, 2, 2, 40, seed=1)
    for c in (small4.ctx, ctx):
        z = np.ones((1, c.n_slots))
        with pytest.raises(binding.EnsiError, match="code -5"):
            c.ct_alloc(1 << 30, c.L)
        c.encode(z, c.L).free()
        sk, pk = c.keygen(None, None, 3)
        pt = c.encode(z, c.L)
        with pytest.raises(binding.EnsiError, match="code -5"):
            c.ct_alloc(1 << 30, c.L)
        ct = c.encrypt(pk, pt)
        with pytest.raises(binding.EnsiError, match="code -5"):
            c.ct_alloc(1 << 30, c.L)
        assert np.abs(c.decrypt(sk, ct) - z).max() < 1e-3
        for h in (ct, pt, pk, sk):
            h.free()
    ctx.close()


@pytest.mark.parametrize("params", [SMALL4, (12, 50, 4, 60, 2, 2, 40)], ids=["1K", "4K"])
def test_matmul_of_wrapped_batches_at_odd_words(params):
    """Wrapped memory is aligned to a word and no more: input and output one word off a 16-byte boundary."""
    import torch
    p = Pair(params)
    s, d, m = p.n // 4, 6, 70
    _, g_gk = p.galois_keys([s, 2 * s, 3 * s])
    W = wl.ternary_weights(np.random.default_rng(8), d, m)
    _, g_ct = p.encrypt_both(wl.pack_columns(p.rng.uniform(-1, 1, (s, d)), p.n), p.pr.L)
    want = p.ctx.ternary_matmul(g_gk, g_ct, s, d, W, "diagonal")
    words = 2 * p.pr.L * p.N
    bufs = [torch.zeros(n * words + 2, dtype=torch.int64, device="cuda") for n in (g_ct.n, m)]
    bufs[0][1:-1] = torch.from_numpy(g_ct.export().reshape(-1).view(np.int64)).cuda()
    torch.cuda.synchronize()
    ct_in, ct_out = (p.ctx.ct_wrap(b[1:].data_ptr(), n, p.pr.L, g_ct.scale) for b, n in zip(bufs, (g_ct.n, m)))
    p.ctx.ternary_matmul(g_gk, ct_in, s, d, W, "diagonal", ct_out)
    assert np.array_equal(ct_out.export(), want.export())
    assert [int(bufs[1][i]) for i in (0, -1)] == [0, 0]
    for h in (g_ct, want, ct_in, ct_out, g_gk):
        h.free()
    p.close()


def test_trim_gives_kept_memory_back_to_the_card(tiny):
    import torch
    ct = tiny.ctx.ct_alloc((200 << 20) // (2 * tiny.pr.L * 8 * tiny.N), tiny.pr.L)
    ct.free()
    before = torch.cuda.mem_get_info()[0]
    tiny.ctx.trim()
    assert torch.cuda.mem_get_info()[0] - before > 190 << 20
    tiny.ctx.trim()  # nothing left to give


def test_full_ring_rotate_batch_longer_than_one_group(full):
    """More ciphertexts than the library raises at once (groups of 64), at a low level to keep the oracle quick."""
    p = full
    n_ct = 67
    steps = [1 if i % 2 else -1 for i in range(n_ct)]
    o_gks, g_gk = p.galois_keys([1, -1])
    z = p.rng.uniform(-1, 1, (n_ct, p.n))
    o_cts, g_ct = p.encrypt_both(z, 2)
    out = p.ctx.rotate(g_gk, g_ct, steps)
    got = out.export()
    for i in (0, 1, 62, 63, 64, 65, 66):
        assert np.array_equal(got[i], p.o.rotate(o_cts[i], o_gks[steps[i]]).limbs()), i
    out.free()
    g_ct.free()
    g_gk.free()
