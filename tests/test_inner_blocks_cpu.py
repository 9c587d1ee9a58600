"""How the rotations of a call are divided among the blocks of the inner product: no wave without a rotation where there are few."""
import simhip

BODY = """
ctx = binding.Context(12, 36, 3, 37, 1, 1, 30, seed=1)
s = ctx.n_slots // 64
fill = ctx.fill_steps(1, ctx.n_slots)
sk, pk = ctx.keygen(None, None, 3)
gk = ctx.galois_keygen(sk, sorted(set(fill) | {r * s for r in range(1, 64)}), None, 4)
masks = ctx.one_hot_masks(1, 3)
for n in (1, 5, 31, 33):
    ct, out = ctx.ct_alloc(n, 3), ctx.ct_alloc(n, 2)
    mark("groups-%d" % n)
    ctx.replicate(gk, ct, list(range(n)), masks, [0] * n, out)
for cols in (5, 32, 34, 64):
    wt = ctx.weights_prepare(np.ones((cols, 8), dtype=np.int8), s, cols, "zero", 3)
    ct, out = ctx.ct_alloc(1, 3), ctx.ct_alloc(8, 3)
    mark("shared-%d" % (cols - 1))
    ctx.ternary_matmul_prepared(gk, ct, wt, out)
for n in (40, 65):
    ct, out = ctx.ct_alloc(n, 3), ctx.ct_alloc(n, 3)
    mark("single-%d" % n)
    ctx.rotate(gk, ct, np.full(n, s, dtype=np.int32), out)
mark("end-0")
"""


def test_few_rotations_take_a_block_each(tmp_path):
    form, n, seen = None, 0, set()
    for c in simhip.run(tmp_path, BODY):
        if c[0] == "mark":
            form, n = c[1].split("-")[0], int(c[1].split("-")[1])
        elif c[0] == "launch" and "k_ks16_innerILi0" in c[2] and form:
            blocks, waves, lds = int(c[3]), int(c[4]) // 64, int(c[5])
            tiles = 4 * 4  # four rows a wave, 16 rows a limb, 3 + 1 limbs
            assert blocks == tiles * -(-n // waves) and lds == waves * 9728, c
            assert waves == (1 if form == "single" or n < 32 else 4), (form, n, waves)
            seen.add((form, n))
    assert seen == {("groups", 1), ("groups", 5), ("groups", 31), ("groups", 33), ("shared", 4), ("shared", 31), ("shared", 33), ("shared", 63), ("single", 40), ("single", 65)}, seen
