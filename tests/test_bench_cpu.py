"""No-GPU checks of the benchmark's host logic: the algorithmic byte / operation counts behind the roofline
entries, for every workload shape, against counts written out by hand."""
import glob
import os
import re

import bench
import workloads as wl


def test_every_workload_has_a_roofline_entry_for_each_kernel_class():
    classes = ["ks_modup_fcols", "ks_frows", "ks_inner", "ks_icols_moddown", "byte_planes", "pm_fcols", "pm_rows_mac", "pm_frows",
               "pm_mac", "pm_irows", "pm_icols_last", "pm_icols_rescale"]
    timers = set()
    for path in glob.glob(os.path.join(bench.ROOT, "paper_2509_09424_amd", "csrc", "*.h*")):
        for line in open(path):
            timers |= set(re.findall(r'"(\w+)"', line)) if "ScopedTimer" in line else set()
    assert set(classes) <= timers  # a class that no launcher times would never be reported
    for w in wl.WORKLOADS:
        if w.log_n != 16:
            continue
        for c in classes:
            dom, roof = bench.roofline_for(w, {c: (1.0, 1)})
            assert dom == c and roof["bound"] == "hbm" and roof["peak"] == 8000.0
            assert roof["achieved"] >= 0.0 and abs(roof["frac"] - roof["achieved"] / 8000.0) < 1e-12


def test_key_switch_counts_of_the_microbenchmark():
    w = wl.BY_NAME["keyswitch"]  # 64 rotations, L = 10, K = 3, alpha = 3 -> beta = 4, ext = 13
    unit = 8.0 * w.N
    _, roof = bench.roofline_for(w, {"ks_modup_fcols": (1.0, 1)})
    assert abs(roof["achieved"] - 64 * (2 * 10 + 4 * 13 + 10) * unit / 1e-3 / 1e9) < 1e-6  # c1 and c0 in, digits and P*c0 out
    _, roof = bench.roofline_for(w, {"ks_frows": (1.0, 1)})
    assert roof["achieved"] == 0.0  # every raise serves one rotation: its row passes are run by the inner product
    _, roof = bench.roofline_for(w, {"ks_inner": (2.0, 1)})
    units = 64 * (4 * 13 + 10 + 2 * 13) + 64 * 2 * 4 * 13  # digits, P*c0, accumulators; one key per rotation
    assert abs(roof["achieved"] - units * unit / 2e-3 / 1e9) < 1e-6
    assert bench.stagewise_rotation_units(w) == 486


def test_matrix_core_operation_count():
    w = wl.BY_NAME["ffn2560"]
    _, roof = bench.roofline_for(w, {"accumulate_mfma": (100.0, 9)})
    # outputs x operands x limb words x byte planes; the second layer runs after the rescale, at 15 limbs
    ops = 2.0 * (2560 * 6912 * 2 * 16 + 6912 * 2560 * 2 * 15) * 65536 * 7
    assert roof["bound"] == "mfma" and roof["peak"] == 5000.0
    assert abs(roof["achieved"] - ops / 0.1 / 1e12) < 1e-6 and roof["launches"] == 9
    assert roof["frac"] == roof["frac_dense"] and abs(roof["frac_own_work"] - 0.6 * roof["frac_dense"]) < 1e-12
    # every operand read once, every output written once: (2560 + 6912) ciphertexts at 16 limbs, (6912 + 2560) at 15
    assert abs(roof["algorithmic_bytes_per_launch"] * 9 - (9472 * 2 * 16 + 9472 * 2 * 15) * 8.0 * 65536) < 1.0
    w = wl.BY_NAME["attn2560"]
    _, roof = bench.roofline_for(w, {"accumulate_mfma": (50.0, 3)})
    assert abs(roof["achieved"] - 2.0 * 2560 * 2560 * 2 * 16 * 65536 * 7 / 0.05 / 1e12) < 1e-6


def test_sums_in_one_kernel_are_the_dominant_one_where_they_are():
    """The 2^12 workload forms its digits where it multiplies them: named, and counted like the contraction of planes."""
    w = wl.BY_NAME["tiny"]
    dom, roof = bench.roofline_for(w, {"accumulate_direct": (0.02, 2), "ks_inner": (0.01, 2)})
    assert dom == roof["kernel"] == "accumulate_direct" and roof["bound"] == "mfma" and roof["launches"] == 2
    assert abs(roof["achieved"] - 2.0 * 64 * 64 * 2 * 3 * 4096 * 5 / 2e-5 / 1e12) < 1e-6
    assert bench.roofline_for(w, {"accumulate_direct": (0.02, 2), "ks_inner": (0.03, 2)})[0] == "ks_inner"


def test_profile_facts_come_from_the_tracked_summary_or_not_at_all(tmp_path, monkeypatch):
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.profile_facts("ffn2560", "accumulate_mfma") == {}
    (tmp_path / "profiles").mkdir()
    (tmp_path / "profiles" / "bench_ffn2560_kernels_and_hbm_counters.txt").write_text(
        "# text\n@facts accumulate_mfma code=%s fetch_GiB_per_step=10.5 write_GiB_per_step=2 mfma_busy=0.6\n@facts other fetch_GiB_per_step=1\n" % bench.code_id())
    f = bench.profile_facts("ffn2560", "accumulate_mfma")
    assert f == {"fetch_GiB_per_step": 10.5, "write_GiB_per_step": 2.0, "mfma_busy": 0.6}
    _, roof = bench.roofline_for(wl.BY_NAME["ffn2560"], {"accumulate_mfma": (100.0, 5)})
    assert abs(roof["traffic"] - 12.5 * 2 ** 30 / 5) < 1e-3 and roof["mfma_busy"] == 0.6 and roof["valu_util"] is None


def test_profile_facts_of_other_code_are_not_reported(tmp_path, monkeypatch):
    csrc = tmp_path / "paper_2509_09424_amd" / "csrc"
    csrc.mkdir(parents=True)
    (tmp_path / "paper_2509_09424_amd" / "build.py").write_text("FLAGS = []\n")
    kernel = csrc / "kernel.hip"
    here = lambda: bench.code_id(str(tmp_path / "paper_2509_09424_amd"))  # noqa: E731
    kernel.write_text("int f(int x) { return x; }\n")
    taken = here()
    kernel.write_text("// what f is for\nint f(int x) {\n    return x;  /* the same */\n}\n")
    assert here() == taken  # comments and layout do not count
    kernel.write_text("int f(int x) { return x + 1; }\n")
    assert here() != taken
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    (tmp_path / "profiles").mkdir()
    for code in ("", "code=%s " % taken):
        (tmp_path / "profiles" / "bench_ffn2560_kernels_and_hbm_counters.txt").write_text("@facts accumulate_mfma %smfma_busy=0.6\n" % code)
        assert bench.profile_facts("ffn2560", "accumulate_mfma") == {}


def test_plaintext_multiplication_counts():
    w = wl.BY_NAME["merge1536"]  # 1536 products into 96 outputs at 16 limbs
    unit = 8.0 * w.N
    _, roof = bench.roofline_for(w, {"pm_rows_mac": (1.0, 3)})
    assert abs(roof["achieved"] - (1536 + 96) * 2 * 16 * unit / 1e-3 / 1e9) < 1e-6
    w = wl.BY_NAME["rope1536"]  # 96 ciphertexts: 3 products each, 2 rotations sharing one raise
    _, roof = bench.roofline_for(w, {"pm_fcols": (1.0, 3)})
    assert abs(roof["achieved"] - 3 * 96 * 4 * 16 * unit / 1e-3 / 1e9) < 1e-6
    _, roof = bench.roofline_for(w, {"ks_modup_fcols": (1.0, 3)})
    assert abs(roof["achieved"] - 96 * (2 * 16 + 4 * 20 + 16) * unit / 1e-3 / 1e9) < 1e-6


def test_giant_and_baby_step_counts():
    w = wl.BY_NAME["ccmmqkbsgs"]  # 96 segments and 1536 elements at period 16, blocks of 2048; 16 + 4 limbs, alpha 4
    assert bench.fill_counts(16, 2048) == (10, 4) and bench.fill_counts(1, 16) == (6, 2)
    unit = 8.0 * w.N
    _, roof = bench.roofline_for(w, {"ks_modup_fcols": (1.0, 1)})
    # raises: 96 inputs at 16 limbs; per segment 4 fill groups and one for its baby rotations at 15; per element 2 and per output 1 at
    # 14; each reads two polynomials and writes four digits over four more limbs, and P*c0
    raises = 96 * (3 * 16 + 4 * 20) + 96 * (4 + 1) * (3 * 15 + 4 * 19) + (1536 * 2 + 16) * (3 * 14 + 4 * 18)
    assert abs(roof["achieved"] - raises * unit / 1e-3 / 1e9) < 1e-6
    _, roof = bench.roofline_for(w, {"ks_frows": (1.0, 1)})
    # of these, the ones that serve several rotations: not the last doubling of a segment's fill, not the relinearisations
    rows = 96 * 2 * (4 * 20 + 16) + 96 * (3 + 1) * 2 * (4 * 19 + 15) + 1536 * 2 * 2 * (4 * 18 + 14)
    assert abs(roof["achieved"] - rows * unit / 1e-3 / 1e9) < 1e-6
    _, roof = bench.roofline_for(w, {"pm_fcols": (1.0, 1)})
    assert abs(roof["achieved"] - (96 * 4 * 16 + 1536 * 4 * 15) * unit / 1e-3 / 1e9) < 1e-6
    w = wl.BY_NAME["ccmmav"]  # one column of V: 32 segments, 512 elements
    _, roof = bench.roofline_for(w, {"ks_icols_moddown": (1.0, 1)})
    # switch-backs at 16, 15 and 14 limbs: accumulators over four more limbs in, ciphertext out
    switches = 32 * (4 * 16 + 8) + (32 * 4 + 512) * (4 * 15 + 8) + (512 * 2 + 1) * (4 * 14 + 8)
    assert abs(roof["achieved"] - switches * unit / 1e-3 / 1e9) < 1e-6


def test_segment_form_counts():
    w = wl.BY_NAME["ccmmqkseg"]  # 96 ciphertexts of K and of Q, period 64 in baby steps of 4: 127 diagonals, 32 giant steps
    assert (w.period, w.baby, w.d_out) == (64, 4, 64) and bench.fill_counts(64, 2048) == (7, 3)
    unit = 8.0 * w.N
    _, roof = bench.roofline_for(w, {"ks_icols_moddown": (1.0, 1)})
    # aligning rotations; fill groups and baby steps of K's operands, relinearisations, giant steps of 123 sums (Q's columns are moved outside)
    switches = 96 * (4 * 16 + 8) + (96 * 3 + 96 * 3 + 127 + 123) * (4 * 15 + 8)
    assert abs(roof["achieved"] - switches * unit / 1e-3 / 1e9) < 1e-6
    _, roof = bench.roofline_for(w, {"pm_fcols": (1.0, 1)})  # 96 head-mask sources at 16 limbs, the 127 diagonals at 14 (each once)
    assert abs(roof["achieved"] - (96 * 4 * 16 + 127 * 4 * 14) * unit / 1e-3 / 1e9) < 1e-6
    _, roof = bench.roofline_for(w, {"pm_rows_mac": (1.0, 1)})  # the 96 head-mask products, term by term
    assert abs(roof["achieved"] - (96 + 96) * 2 * 16 * unit / 1e-3 / 1e9) < 1e-6
    # the 6112 sorting products of 127 diagonals into 64 columns, source by source: row passes of each diagonal and each column
    for name, units in (("pm_frows", 127 * 4 * 14), ("pm_mac", (127 + 64) * 2 * 14), ("pm_irows", 64 * 4 * 14)):
        _, roof = bench.roofline_for(w, {name: (1.0, 1)})
        assert abs(roof["achieved"] - units * unit / 1e-3 / 1e9) < 1e-6
    # library transforms of the products: 96 * 4 operands (two polynomials of 15 limbs, two passes, in and out), 127 x 3 sums back
    _, roof = bench.roofline_for(w, {"ntt_fwd_cols": (1.0, 1)})
    assert abs(roof["achieved"] - 4 * (96 * 4 * 2 * 15 + 127 * 3 * 15) * unit / 1e-3 / 1e9) < 1e-6
    w = wl.BY_NAME["ccmmavseg"]  # one column of V, 8 segments of 64 tokens, baby steps of 8: 16 giant steps
    assert (w.period, w.baby) == (64, 8)
    _, roof = bench.roofline_for(w, {"ks_modup_fcols": (1.0, 1)})
    # raises: the column at 16 limbs; per segment 3 fill groups and one for its baby steps, the 16 relinearisations and the 15 giant steps
    # of the sums, at 15
    assert abs(roof["achieved"] - (1 * (3 * 16 + 4 * 20) + (8 * 4 + 16 + 15) * (3 * 15 + 4 * 19)) * unit / 1e-3 / 1e9) < 1e-6
