"""The two streams of ensi_encrypt: what may run at the same time, within a call and after one that failed."""
import pytest

import simhip

BODY = """
ctx = binding.Context(12, 50, 2, 60, 1, 1, 40, seed=1)
N = ctx.N
sk, pk = ctx.keygen(None, None, 3)
few, many = [ctx.pt_import(np.zeros((n, N), dtype=np.int64), 2) for n in (8, 600)]
zero = np.zeros((600, N), dtype=np.int8)
ct = ctx.ct_alloc(600, 2)
slots = np.zeros((600, N // 2))
call = {"encrypt": lambda: ctx.encrypt(pk, many, zero, zero, zero), "encode": lambda: ctx.encode(slots, 2), "decrypt": lambda: ctx.decrypt(sk, ct)}["%s"]
mark("first")
sim.simhip_fail_copy(%d)
try:
    call()
    failed = False
except binding.EnsiError:
    failed = True
assert failed == (%d >= 0)
sim.simhip_fail_copy(-1)
mark("second")
ctx.encrypt(pk, few, zero[:8], zero[:8], zero[:8])
mark("end")
"""


def first_and_second(tmp_path, call, fail):
    calls = simhip.run(tmp_path, BODY % (call, fail, fail))
    at = {c[1]: k for k, c in enumerate(calls) if c[0] == "mark"}
    return calls, at, simhip.unordered(calls)


def test_errors_are_copied_beside_the_mask_only(tmp_path):
    """Three chunks of ciphertexts: a chunk's errors may arrive while its own mask is worked on, and not while the chunk before is added."""
    calls, at, pairs = first_and_second(tmp_path, "encrypt", -1)
    ours = [(i, k) for i, k in pairs if at["first"] < i < at["second"] and at["first"] < k < at["second"]]
    adds = [k for k, c in enumerate(calls) if c[0] == "launch" and "k_cl_icols_add" in c[2] and at["first"] < k < at["second"]]
    assert len(adds) == 3 and ours
    for i, k in ours:
        assert calls[k][0] == "copy" and calls[k][1] != "(nil)" and not any(i <= a < k for a in adds), (calls[i], calls[k])


@pytest.mark.parametrize("call,fail", [("encrypt", 1), ("encrypt", 2), ("encrypt", 4), ("encrypt", 5), ("encode", 1), ("decrypt", 0), ("decrypt", 1)])
def test_nothing_of_a_failed_call_runs_beside_the_next(tmp_path, call, fail):
    """A copy fails with kernels enqueued that work on the memory to which the next call copies its errors."""
    calls, at, pairs = first_and_second(tmp_path, call, fail)
    assert any(c[0] == "launch" for c in calls[at["first"]:at["second"]])
    assert any(c[0] == "copy" and c[1] != "(nil)" for c in calls[at["second"]:])
    crossing = [(calls[i], calls[k]) for i, k in pairs if i < at["second"] < k]
    assert not crossing, crossing[:3]


def test_small_batches_keep_to_one_stream(tmp_path):
    """Up to 16 KiB a polynomial a second stream costs more than it hides; whole calls at both sides of the line."""
    calls = simhip.run(tmp_path, """
ctx = binding.Context(12, 36, 3, 37, 1, 1, 30, seed=1)
sk, pk = ctx.keygen(None, None, 3)
pts = [ctx.pt_import(np.zeros((n, ctx.N), dtype=np.int64), 3) for n in (4, 5)]
zero = np.zeros((5, ctx.N), dtype=np.int8)
for n, pt in zip((4, 5), pts):
    mark("%d" % n)
    ctx.encrypt(pk, pt, zero[:n], zero[:n], zero[:n])
mark("end")
""")
    at = {c[1]: k for k, c in enumerate(calls) if c[0] == "mark"}
    streams = [{c[1] for c in calls[at[a]:at[b]] if c[0] in ("copy", "launch")} for a, b in (("4", "5"), ("5", "end"))]
    assert [len(s) for s in streams] == [1, 2] and not any(c[0] in ("record", "wait") and c[1] != "(nil)" for c in calls[at["4"]:at["5"]])
    assert not [p for p in simhip.unordered(calls) if at["4"] < p[1] < at["5"]]
