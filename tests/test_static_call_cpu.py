"""The allocation-free rotation: kernels and nothing else, its descriptors among their arguments."""
import simhip


def test_rotate_static_enqueues_kernels_only(tmp_path):
    calls = simhip.run(tmp_path, """
ctx = binding.Context(12, 36, 3, 37, 1, 1, 30, seed=1)
sk, pk = ctx.keygen(None, None, 3)
gk = ctx.galois_keygen(sk, [1], None, 4)
for n in (64, 1):
    ct, out = ctx.ct_alloc(n, 3), ctx.ct_alloc(n, 3)
    mark("begin")
    ctx.rotate_static(gk, ct, np.ones(n, dtype=np.int32), out)
    mark("end")
""")
    marks = [k for k, c in enumerate(calls) if c[0] == "mark"]
    for a, b in zip(marks[::2], marks[1::2]):
        what = calls[a + 1:b]
        assert what and {c[0] for c in what} == {"launch"} and "k_upload" in what[0][2], what
