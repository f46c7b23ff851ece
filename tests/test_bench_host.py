"""Host logic of bench.py (no GPU): the per-launch work that the per-kernel
table divides by each kernel's time, with and without the rotated pre-pass
of the Eq. 3 bound."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import bench  # noqa: E402


def _stats(prepass, rebound_items, rebound_pairs):
    return [{"thresh_pairs": 1.0e9, "refine_pairs": 0.0, "count_pairs": 5.0e8,
             "bound_pairs": 6.0e9, "rebound_pairs": rebound_pairs,
             "prepass_dprime": prepass, "rebound_items": rebound_items,
             "cand_listed": 1.0e6}]


def test_bound_work_with_prepass():
    n, m, d = 20000, 3000, 200
    prof = [("k_bound", 1, 8.0), ("k_bound/rebound", 1, 4.0), ("k_aug_ident", 2, 1.0)]
    t = bench.kernel_table(prof, _stats(62, 500, 2.0e9), 1, n, m, d, 10, "fp32")
    # the pre-pass: d' + 2 = 64 terms per pair; the second bound: d + 2
    assert t["k_bound"]["work_per_launch"] == 2.0 * 64 * 6.0e9
    assert t["k_bound/rebound"]["work_per_launch"] == 2.0 * 202 * 2.0e9
    # identity rows: every user and the 500 re-bounded items, 224 BF16
    # values written per row (d + 2 rounded up to 32 past 176 terms)
    rows = n + 500
    assert t["k_aug_ident"]["work_per_launch"] == (rows * 4.0 * d + rows * 2.0 * 224) / 2
    assert abs(t["k_bound"]["achieved"] - 2.0 * 64 * 6.0e9 / 8.0e-3 / 1e12) < 1e-9


def test_bound_work_without_prepass():
    n, m, d = 20000, 3000, 100
    prof = [("k_bound", 1, 8.0), ("k_aug_ident", 2, 1.0)]
    t = bench.kernel_table(prof, _stats(0, 0, 0.0), 1, n, m, d, 10, "bf16")
    assert t["k_bound"]["work_per_launch"] == 2.0 * 102 * 6.0e9
    mpad = (m + 63) // 64 * 64
    assert t["k_aug_ident"]["work_per_launch"] == ((n + m) * 4.0 * d + (n + mpad) * 2.0 * 112) / 2
    assert "k_bound/rebound" not in t


def test_selection_work_under_either_name():
    # the selection has the name of the kernel that ran; its bytes are the
    # lists' entries and a threshold per user
    n, m, d = 20000, 3000, 100
    prof = [("k_thresh_select/main", 2, 1.0), ("k_thresh_final/main", 1, 1.0)]
    t = bench.kernel_table(prof, _stats(0, 0, 0.0), 1, n, m, d, 10, "fp8")
    assert t["k_thresh_select/main"]["work_per_launch"] == 12.0 * (1.0e6 + n) / 2
    assert t["k_thresh_final/main"]["work_per_launch"] == 12.0 * (1.0e6 + n)


def test_result_line_is_short():
    # forty kernels in the table and in each of four variants: one JSON line of
    # less than 6 KB with the contract's keys, values to six digits
    import json
    k = {f"k_some_long_kernel_name_{i}/main": {
        "launches_per_step": 1.0 / 3, "ms_per_step": 10.0 / (i + 3), "ms_per_launch": 1.0 / 7,
        "bound": "mfma", "unit_work": "flop", "work_per_launch": 1e12 / 3, "achieved": 1e3 / 3,
        "peak": 2500.0, "rate_unit": "TFLOP/s", "frac": 1.0 / 3} for i in range(40)}
    out = {"metric": "m", "value": 2576.123456789, "unit": "G pairs/s", "n_gpus": 1, "steps": 20,
           "warmup": 5, "ms_per_step": 77.6 / 3, "higher_is_better": True, "scaling": "weak",
           "vs_baseline": None, "dtype": "fp32", "data": "synthetic", "config": {"n": 2000000},
           "kernels": k, "paper_context": "x" * 300, "top_ids": list(range(10 ** 5, 10 ** 5 + 20)),
           "variants": {v: {"ms_per_step": 1 / 3, "value": 2e3 / 3, "same_top_n": True, "kernels": k,
                            "dominant_kernel": "k_thresh_screen/main", "dominant_frac": 1 / 3,
                            "recheck_pairs": 1e8 / 3, "cand_listed": 1e8 / 3, "cand_pairs": 1e7 / 3,
                            "refine_users": 0.0} for v in ("bf16", "fp8", "fp6", "fp4")}}
    line = bench.result_line(out)
    assert "\n" not in line and len(line) < 6000
    got = json.loads(line)
    for key in ("metric", "unit", "n_gpus", "steps", "warmup", "higher_is_better", "scaling",
                "vs_baseline", "dtype", "data", "config"):
        assert got[key] == out[key]
    assert abs(got["value"] - out["value"]) <= 1e-5 * out["value"]
    assert abs(got["ms_per_step"] - out["ms_per_step"]) <= 1e-5 * out["ms_per_step"]
    assert got["variants"]["fp8"]["same_top_n"] and "kernels" not in got["variants"]["fp8"]
    top = max(k, key=lambda a: k[a]["ms_per_step"])
    assert got["kernels"][top]["ms_per_step"] == 3.33333
