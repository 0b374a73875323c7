"""More than eight strips of 16 output channels for every compute unit at M <= 16: which kernel takes them (half the strips per
workgroup of slice_kernel, or all of them in one of column_kernel), on both sides of every line, and the results there."""

import pytest

import paper_2510_16045_amd as ams
from oracle import ams_oracle as O
from paper_2510_16045_amd import synth
from test_gpu_slice_kernel import PAIRS, REC_K, check, dev, problem, scales_per_run

torch = pytest.importorskip("torch")

# (format, M, N, records, entry, kernel)
LINES = [
    # one scale per row, side groups
    ("FP425", 1, 40005, 63, "plain", "slice"), ("FP425", 1, 40005, 64, "plain", "column"), ("FP425", 2, 40005, 64, "plain", "slice"), ("FP425", 1, 65552, 64, "plain", "slice"),
    ("FP425", 8, 128256, 3, "plain", "slice"), ("FP433", 6, 65531, 1, "plain", "slice"), ("FP45", 5, 40005, 22, "plain", "column"), ("FP45", 5, 40005, 23, "plain", "slice"),
    ("FP6", 8, 40005, 26, "plain", "slice"), ("FP6", 2, 65552, 2, "plain", "column"), ("FP6", 2, 65552, 3, "plain", "slice"),
    # none
    ("FP533", 1, 40960, 3, "plain", "slice"), ("FP533", 1, 40960, 2, "plain", "column"), ("FP533", 4, 40976, 20, "plain", "column"), ("FP5", 8, 33000, 7, "plain", "slice"),
    ("FP4", 3, 98304, 5, "plain", "slice"), ("FP4", 3, 98320, 5, "plain", "column"), ("FP533", 2, 131072, 5, "plain", "column"),
    # 9 to 16 rows
    ("FP425", 9, 40005, 64, "plain", "slice"), ("FP45", 16, 40005, 63, "plain", "column"),
    # one scale per run
    ("FP533", 1, 40005, 3, "grouped", "slice"), ("FP533", 2, 40005, 2, "grouped", "column"), ("FP6", 8, 40005, 8, "grouped", "slice"), ("FP433", 5, 40005, 7, "grouped", "column"),
    ("FP533", 8, 50000, 24, "grouped", "slice"), ("FP533", 1, 50000, 23, "grouped", "column"), ("FP4", 6, 50000, 24, "grouped", "slice"), ("FP5", 6, 50000, 23, "grouped", "column"),
    ("FP425", 1, 65536, 64, "grouped", "slice"), ("FP425", 1, 65536, 63, "grouped", "column"), ("FP5", 8, 65536, 64, "grouped", "column"), ("FP425", 16, 40005, 63, "grouped", "column"),
]


def plan_of(name, M, N, n_rec, entry):
    fmt = getattr(ams, name)
    K = REC_K[fmt] * n_rec - 8 * (n_rec % 3)  # the last record whole, or 8 or 16 channels short
    return fmt, K, ams.ams_linear_plan(fmt, M, N, K, with_workspace={"plain": 0, "grouped": 2}[entry])


@pytest.mark.parametrize("name,M,N,n_rec,entry,kernel", LINES)
def test_which_kernel(name, M, N, n_rec, entry, kernel):
    plan = plan_of(name, M, N, n_rec, entry)[2]
    strips = min(16, -(-(-(-N // 16)) // 256))
    assert plan.startswith(kernel + " ") and f"strips_per_wg={(strips + 1) // 2 if kernel == 'slice' else strips} " in plan, plan


@pytest.mark.gpu
@pytest.mark.parametrize("name,M,N,n_rec,entry,kernel", LINES)
def test_results_on_both_sides(name, M, N, n_rec, entry, kernel):
    fmt, K, plan = plan_of(name, M, N, n_rec, entry)
    ofmt = dict(PAIRS)[fmt]
    codes, scales, rows = problem(fmt, ofmt, N, K, N + n_rec)
    X = synth.activations(M, K, 50 + M)
    packed, x = dev(ams.ams_pack_codes(fmt, codes)), dev(X)
    if entry == "grouped":
        scales, run_packed = scales_per_run(N, K, REC_K[fmt], n_rec)
        y = ams.ams_linear_grouped(packed, dev(run_packed), REC_K[fmt], x, N, fmt)
        ref = O.linear(codes[rows], scales[rows], X, ofmt, REC_K[fmt])
    else:
        y, ref = ams.ams_linear(packed, dev(scales), x, N, fmt), O.linear(codes[rows], scales[rows], X, ofmt)
    check(y, ref, rows, f"{name} N={N} K={K} M={M} {entry}: {plan}")
