"""The kernel that streams the activations beside the weights (slice plans): every number of
strips per workgroup, every count of staged rows, wavefronts with no, one and many records, channels
beyond K inside the last record, ragged last strips and workgroups, and K split over workgroups; sampled
rows against the oracle.  One activation row of infinities must leave the others alone."""

import numpy as np
import pytest

import paper_2510_16045_amd as ams
from oracle import ams_oracle as O
from paper_2510_16045_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

PAIRS = [(ams.FP533, O.FP533), (ams.FP425, O.FP425), (ams.FP45, O.FP45), (ams.FP433, O.FP433), (ams.FP6, O.FP6_E2M3), (ams.FP5, O.FP5_E2M2), (ams.FP4, O.FP4_E2M1)]
REC_K = {ams.FP533: 96, ams.FP425: 128, ams.FP45: 128, ams.FP433: 96, ams.FP6: 96, ams.FP5: 128, ams.FP4: 128}


def dev(a):
    return torch.from_numpy(a.view(np.int16)).cuda().view(torch.float16) if a.dtype == np.float16 else torch.from_numpy(a).cuda()


def problem(fmt, ofmt, N, K, seed):
    rng = np.random.default_rng(seed)
    codes = rng.integers(0, 1 << ofmt.code_bits, size=(N, K), dtype=np.uint8)
    codes = (codes & 0xFE) | np.repeat(codes[:, :: ofmt.group] & 1, ofmt.group, axis=1)[:, :K]
    scales = rng.uniform(0.001, 0.01, size=N).astype(np.float16)
    n_strips = -(-N // 16)
    strips = np.unique(np.r_[0, 1, n_strips - 2, n_strips - 1, np.arange(3, n_strips, max(1, n_strips // 9))])
    strips = strips[(strips >= 0) & (strips < n_strips)]
    rows = np.concatenate([np.arange(16 * t, min(N, 16 * t + 16)) for t in strips])
    return codes, scales, rows


def check(y, ref, rows, what, keep=slice(None)):
    # fp32 sums rounded to fp16 once: at most 2^-11 per output, 1e-3 as in the other parity tests
    y = y.cpu().view(torch.int16).numpy().view(np.float16).astype(np.float64)[:, rows][keep]
    assert np.all(np.isfinite(y)), what
    assert np.linalg.norm(y - ref[keep]) <= 1e-3 * np.linalg.norm(ref[keep]), what


@pytest.mark.parametrize("fmt,ofmt", PAIRS)
@pytest.mark.parametrize("spw", range(1, 9))
def test_strips_rows_and_records(fmt, ofmt, spw):
    # N: spw strips per workgroup, the last workgroup short and its last strip ragged
    N = 16 * (256 * (spw - 1) + 130) - 5 if spw > 1 else 16 * 130 - 5
    rec = REC_K[fmt]
    # records per strip: 1, 3 (some wavefronts have none), 8, 17, and one more record that ends after 8 channels
    for n_rec, Ms in ((1, (1, 32)), (3, (3, 17)), (8, (4, 9)), (17, (1, 8, 16, 32)), (34, (2, 5))):
        K = rec * (n_rec - 1) + (8 if n_rec in (3, 34) else rec - 8 if n_rec == 17 else rec)
        codes, scales, rows = problem(fmt, ofmt, N, K, 100 * spw + n_rec)
        wp, sc = dev(ams.ams_pack_codes(fmt, codes)), dev(scales)
        for M in Ms:
            plan = ams.ams_linear_plan(fmt, M, N, K)
            few = (spw == 8 and n_rec <= 16) or (spw in (6, 7) and n_rec == 1)  # at M > 16 those are column_kernel's
            assert plan.startswith("column " if M > 16 and few else "slice ") and f"strips_per_wg={spw} " in plan, plan
            X = synth.activations(M, K, 70 + M)
            ref = O.linear(codes[rows], scales[rows], X, ofmt)
            what = f"{ofmt.name} N={N} K={K} M={M}: {plan}"
            x = dev(X)
            check(ams.ams_linear(wp, sc, x, N, fmt), ref, rows, what)
            if M > 2 and n_rec in (3, 17):
                x[M // 2] = float("inf")
                check(ams.ams_linear(wp, sc, x, N, fmt), ref, rows, "beside a row of infinities: " + what, [m for m in range(M) if m != M // 2])


def test_plans_are_the_ones_meant():
    for spw in range(1, 9):
        N = 16 * (256 * (spw - 1) + 130) - 5 if spw > 1 else 16 * 130 - 5
        for M in (3, 5, 9, 16):
            for fmt in (ams.FP533, ams.FP425, ams.FP433):
                plan = ams.ams_linear_plan(fmt, M, N, 17 * REC_K[fmt] - 8)
                assert plan.startswith("slice ") and f"strips_per_wg={spw} " in plan, plan


@pytest.mark.parametrize("fmt,ofmt", PAIRS)
@pytest.mark.parametrize("N,K,Ms", [(2560, 9728, (4, 8, 16, 32)), (4091, 14336, (8, 32)), (5120, 12808, (5, 17))])
def test_k_split_over_workgroups(fmt, ofmt, N, K, Ms):
    codes, scales, rows = problem(fmt, ofmt, N, K, 7)
    wp, sc = dev(ams.ams_pack_codes(fmt, codes)), dev(scales)
    ws = torch.zeros(16 << 20, dtype=torch.uint8, device="cuda")
    for M in Ms:
        X = synth.activations(M, K, 80 + M)
        ref = O.linear(codes[rows], scales[rows], X, ofmt)
        x = dev(X)
        plan = ams.ams_linear_plan(fmt, M, N, K, with_workspace=True)
        assert plan.startswith("slice ") and ("k_slices=1 " in plan) == (M == 4), plan
        what = f"{ofmt.name} N={N} K={K} M={M}: {plan}"
        first = ams.ams_linear_ws(wp, sc, x, N, fmt, ws)
        check(first, ref, rows, what)
        for _ in range(3):  # the calls leave the workspace ready for the next one, and the result does not change
            assert torch.equal(ams.ams_linear_ws(wp, sc, x, N, fmt, ws), first), what
        assert torch.equal(ams.ams_linear_static_ws(wp, sc, x, N, fmt), first), what
        assert not ws[: 4 * 16384].any(), what


def test_slices_that_do_not_divide_the_records():
    fmt, ofmt, N, K, M = ams.FP533, O.FP533, 1030, 96 * 131 + 8, 16  # 132 records in eight slices
    plan = ams.ams_linear_plan(fmt, M, N, K, with_workspace=True)
    assert plan.startswith("slice ") and "k_slices=8 " in plan, plan
    codes, scales, rows = problem(fmt, ofmt, N, K, 9)
    ws = torch.zeros(16 << 20, dtype=torch.uint8, device="cuda")
    X = synth.activations(M, K, 90)
    y = ams.ams_linear_ws(dev(ams.ams_pack_codes(fmt, codes)), dev(scales), dev(X), N, fmt, ws)
    check(y, O.linear(codes[rows], scales[rows], X, ofmt), rows, "uneven slices")


@pytest.mark.parametrize("fmt,ofmt", PAIRS)
@pytest.mark.parametrize("spw", [1, 2, 3, 5, 7, 8])
def test_one_scale_per_run(fmt, ofmt, spw):
    # runs of one, two and four records, a short last run, ragged last strips and workgroups, all staged row counts
    N = 16 * (256 * (spw - 1) + 130) - 5 if spw > 1 else 16 * 130 - 5
    rec = REC_K[fmt]
    for n_rec, mult, Ms in ((2, 1, (1, 32)), (17, 1, (4, 16, 32)), (18, 2, (3, 8)), (35, 4, (1, 17))):
        K, sg = rec * (n_rec - 1) + 8 * (n_rec % 3 + 1), rec * mult
        codes, _, rows = problem(fmt, ofmt, N, K, 100 * spw + n_rec)
        runs, n_strips = -(-K // sg), -(-N // 16)
        scales = np.random.default_rng(n_rec).uniform(0.001, 0.01, size=(n_strips * 16, runs)).astype(np.float16)
        packed = np.ascontiguousarray(scales.reshape(n_strips, 16, runs).transpose(0, 2, 1))  # [strip][run][row in strip]
        wp, sc = dev(ams.ams_pack_codes(fmt, codes)), dev(packed)
        for M in Ms:
            X = synth.activations(M, K, 60 + M)
            ref = O.linear(codes[rows], scales[rows], X, ofmt, sg)
            plan = ams.ams_linear_plan(fmt, M, N, K, with_workspace=2)
            assert plan.startswith("column " if M > 16 and (spw == 8 and n_rec <= 16 or spw >= 6 and n_rec <= 2) else "slice "), plan
            what = f"{ofmt.name} N={N} K={K} M={M} run={sg}: {plan}"
            x = dev(X)
            check(ams.ams_linear_grouped(wp, sc, sg, x, N, fmt), ref, rows, what)
            if M > 2:
                x[M // 2] = float("inf")
                check(ams.ams_linear_grouped(wp, sc, sg, x, N, fmt), ref, rows, "beside a row of infinities: " + what, [m for m in range(M) if m != M // 2])


def scales_per_run(N, K, sg, seed):
    """[rows padded to strips, runs] and the same in the order the kernels read."""
    runs, n_strips = -(-K // sg), -(-N // 16)
    scales = np.random.default_rng(seed).uniform(0.001, 0.01, size=(n_strips * 16, runs)).astype(np.float16)
    return scales, np.ascontiguousarray(scales.reshape(n_strips, 16, runs).transpose(0, 2, 1))


# (format, M, N, records, entry, kernel): both sides of the lines between slice_kernel and column_kernel on aligned rows
LINES = [
    ("FP433", 4, 48000, 1, "plain", "slice"), ("FP433", 3, 40965, 11, "grouped", "column"), ("FP433", 3, 40965, 16, "grouped", "slice"),
    ("FP45", 4, 65536, 2, "plain", "column"), ("FP45", 4, 65531, 3, "plain", "slice"), ("FP6", 3, 128251, 1, "plain", "column"), ("FP6", 3, 128256, 3, "plain", "slice"),
    ("FP425", 4, 65531, 1, "grouped", "column"), ("FP425", 3, 57339, 24, "grouped", "slice"), ("FP533", 3, 65536, 15, "grouped", "column"),
    ("FP533", 4, 128251, 2, "grouped", "column"), ("FP533", 4, 128251, 3, "grouped", "slice"), ("FP4", 4, 65531, 9, "grouped", "column"),
    ("FP533", 17, 32787, 79, "plain", "column"), ("FP533", 17, 32787, 80, "plain", "slice"), ("FP533", 32, 32787, 80, "plain", "slice"), ("FP4", 32, 32787, 80, "plain", "slice"),
    ("FP4", 32, 32763, 16, "plain", "column"), ("FP533", 32, 32763, 17, "plain", "slice"), ("FP5", 32, 28667, 3, "plain", "slice"), ("FP5", 17, 28667, 2, "grouped", "column"),
    ("FP425", 24, 24571, 1, "plain", "column"), ("FP425", 24, 24571, 2, "grouped", "column"), ("FP45", 16, 32763, 2, "plain", "column"),
    ("FP425", 1, 4107, 97, "plain", "column"), ("FP533", 1, 6139, 97, "grouped", "column"), ("FP533", 1, 6139, 96, "plain", "slice"), ("FP6", 1, 7163, 97, "grouped", "column"),
    ("FP5", 2, 7163, 145, "grouped", "column"), ("FP433", 1, 1003, 201, "plain", "column"), ("FP533", 1, 1003, 201, "grouped", "column"), ("FP45", 1, 1003, 250, "grouped", "column"),
    ("FP533", 16, 2555, 198, "ws", "column"), ("FP425", 32, 2043, 200, "ws", "column"), ("FP533", 32, 5115, 100, "ws", "column"), ("FP45", 32, 2043, 200, "ws", "column"),
    ("FP6", 16, 3579, 230, "ws", "column"), ("FP425", 32, 1531, 108, "ws", "column"), ("FP533", 16, 5115, 100, "ws", "slice"),
]


@pytest.mark.parametrize("name,M,N,n_rec,entry,kernel", LINES)
def test_both_sides_of_the_lines(name, M, N, n_rec, entry, kernel):
    fmt = getattr(ams, name)
    ofmt = dict(PAIRS)[fmt]
    K = REC_K[fmt] * n_rec - 8 * (n_rec % 3)  # the last record whole, or 8 or 16 channels short
    plan = ams.ams_linear_plan(fmt, M, N, K, with_workspace={"plain": 0, "ws": 1, "grouped": 2}[entry])
    assert plan.startswith(kernel + " ") and ("k_slices=1 " in plan) == (entry != "ws"), plan
    codes, scales, rows = problem(fmt, ofmt, N, K, N + n_rec)
    X = synth.activations(M, K, 50 + M)
    wp, x = dev(ams.ams_pack_codes(fmt, codes)), dev(X)
    what = f"{name} N={N} K={K} M={M} {entry}: {plan}"
    if entry == "grouped":
        sg = REC_K[fmt]
        scales, packed = scales_per_run(N, K, sg, n_rec)
        call = lambda: ams.ams_linear_grouped(wp, sc, sg, x, N, fmt)
        sc, ref = dev(packed), O.linear(codes[rows], scales[rows], X, ofmt, sg)
    else:
        sc, ref = dev(scales), O.linear(codes[rows], scales[rows], X, ofmt)
        ws = torch.zeros(16 << 20, dtype=torch.uint8, device="cuda")
        call = lambda: ams.ams_linear_ws(wp, sc, x, N, fmt, ws) if entry == "ws" else ams.ams_linear(wp, sc, x, N, fmt)
    first = call()
    check(first, ref, rows, what)
    assert torch.equal(call(), first), what
    if entry == "ws":
        assert torch.equal(ams.ams_linear_static_ws(wp, sc, x, N, fmt), first), what
        assert not ws[: 4 * 16384].any(), what
