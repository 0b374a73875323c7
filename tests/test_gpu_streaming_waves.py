"""slice_kernel where a wavefront asks for more ahead on one strip, and where only twelve of a workgroup's sixteen wavefronts take records (two strips at M <= 4, one strip at 9 to
16 rows): as many records as streaming wavefronts, one fewer, one more, two and four rounds of them, and a wavefront's last
record short; one scale per row, per run, and K split over workgroups; sampled rows against the oracle."""

import numpy as np
import pytest

import paper_2510_16045_amd as ams
from oracle import ams_oracle as O
from paper_2510_16045_amd import synth
from test_gpu_slice_kernel import PAIRS, REC_K, check, dev, problem, scales_per_run

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt,ofmt", PAIRS)
@pytest.mark.parametrize("strips,N,Ms", [(2, 16 * 300 - 5, (1, 4)), (1, 16 * 140 - 5, (9, 12, 15))])
def test_records_around_the_streaming_wavefronts(fmt, ofmt, strips, N, Ms):
    for n_rec in (11, 12, 13, 24, 25, 48, 49):
        K = REC_K[fmt] * n_rec - 8 * (n_rec % 3)
        codes, scales, rows = problem(fmt, ofmt, N, K, n_rec)
        packed = dev(ams.ams_pack_codes(fmt, codes))
        run_scales, run_packed = scales_per_run(N, K, 2 * REC_K[fmt], 4)
        for M in Ms:
            eight = strips == 1 and (n_rec in (24, 25) if REC_K[fmt] == 96 else M == 15 and n_rec >= 18)  # wavefronts, which are the faster there
            plan = ams.ams_linear_plan(fmt, M, N, K)
            assert plan.startswith("slice ") and f"strips_per_wg={strips} " in plan and (" waves=8 " if eight else " waves=16 ") in plan, plan
            X = synth.activations(M, K, 50 + M)
            what = f"{ofmt.name} N={N} K={K} M={M}: {plan}"
            check(ams.ams_linear(packed, dev(scales), dev(X), N, fmt), O.linear(codes[rows], scales[rows], X, ofmt), rows, what)
            y = ams.ams_linear_grouped(packed, dev(run_packed), 2 * REC_K[fmt], dev(X), N, fmt)
            check(y, O.linear(codes[rows], run_scales[rows], X, ofmt, 2 * REC_K[fmt]), rows, "scales per run, " + what)


@pytest.mark.parametrize("fmt,ofmt", PAIRS)
def test_streaming_wavefronts_and_slices_of_k(fmt, ofmt):
    N, K, M = 507, 16392, 15
    plan = ams.ams_linear_plan(fmt, M, N, K, with_workspace=True)
    assert plan.startswith("slice ") and " strips_per_wg=1 " in plan and "k_slices=1 " not in plan and " waves=16 " in plan, plan
    codes, scales, rows = problem(fmt, ofmt, N, K, 6)
    X = synth.activations(M, K, 61)
    packed, sc, x, ws = dev(ams.ams_pack_codes(fmt, codes)), dev(scales), dev(X), torch.zeros(16 << 20, dtype=torch.uint8, device="cuda")
    first = ams.ams_linear_ws(packed, sc, x, N, fmt, ws)
    check(first, O.linear(codes[rows], scales[rows], X, ofmt), rows, plan)
    assert torch.equal(ams.ams_linear_ws(packed, sc, x, N, fmt, ws), first) and not ws[: 4 * 16384].any(), plan


@pytest.mark.parametrize("fmt,ofmt", [p for p in PAIRS if REC_K[p[0]] == 96])
def test_two_records_ahead_on_tiles_of_sixteen_rows(fmt, ofmt):
    # two and three records for a wavefront, one more and one fewer; whole rows of X and rows dealt to two workgroups
    for n_rec, N, M in ((16, 2300, 9), (17, 4096, 16), (23, 16 * 130 - 5, 12), (24, 2000, 26), (25, 16 * 125, 19), (28, 2064, 15)):
        K = 96 * n_rec - 8 * (n_rec % 12)
        plan = ams.ams_linear_plan(fmt, M, N, K)
        assert plan.startswith("slice ") and " x_ahead=2" in plan and " waves=8 " in plan, plan
        codes, scales, rows = problem(fmt, ofmt, N, K, n_rec)
        X = synth.activations(M, K, 90 + M)
        y = ams.ams_linear(dev(ams.ams_pack_codes(fmt, codes)), dev(scales), dev(X), N, fmt)
        check(y, O.linear(codes[rows], scales[rows], X, ofmt), rows, f"{ofmt.name} N={N} K={K} M={M}: {plan}")


@pytest.mark.parametrize("fmt,ofmt", [p for p in PAIRS if REC_K[p[0]] == 128])
def test_two_records_of_activations_ahead(fmt, ofmt):
    # 13 to 16 rows, one scale per row and one per run; 26 rows: dealt to two workgroups
    for n_rec, N, M, run in ((18, 2300, 13, 1), (24, 4096, 15, 4), (25, 16 * 130 - 5, 14, 2), (31, 2000, 26, 8)):
        K, group = 128 * n_rec - 8 * (n_rec % 12), 128 * run
        plan = [ams.ams_linear_plan(fmt, M, N, K, with_workspace=w) for w in (0, 2)]
        assert all(p.startswith("slice ") and " x_ahead=2" in p and " waves=8 " in p for p in plan), plan
        codes, scales, rows = problem(fmt, ofmt, N, K, n_rec)
        run_scales, packed = scales_per_run(N, K, group, n_rec)
        X = synth.activations(M, K, 95 + M)
        w, what = dev(ams.ams_pack_codes(fmt, codes)), f"{ofmt.name} N={N} K={K} M={M}: {plan}"
        check(ams.ams_linear(w, dev(scales), dev(X), N, fmt), O.linear(codes[rows], scales[rows], X, ofmt), rows, what)
        y = ams.ams_linear_grouped(w, dev(packed), group, dev(X), N, fmt)
        check(y, O.linear(codes[rows], run_scales[rows], X, ofmt, group), rows, "scales per run, " + what)


@pytest.mark.parametrize("fmt,ofmt,n_recs", [(ams.FP533, O.FP533, (96, 97, 161)), (ams.FP5, O.FP5_E2M2, (128, 129, 241)), (ams.FP4, O.FP4_E2M1, (96, 111, 161))])
def test_two_records_ahead_on_one_strip(fmt, ofmt, n_recs):
    # whole rounds of sixteen wavefronts and one record more, one row and two, a last record that ends after 8 channels
    for n_rec, Ms, N in zip(n_recs, ((1,), (1,), (1, 2)), (16 * 7, 16 * 219 - 5, 16 * 30 - 5)):
        K = REC_K[fmt] * (n_rec - 1) + (REC_K[fmt] if n_rec == n_recs[0] else 8)
        codes, scales, rows = problem(fmt, ofmt, N, K, n_rec)
        packed = dev(ams.ams_pack_codes(fmt, codes))
        for M in Ms:
            plan = ams.ams_linear_plan(fmt, M, N, K)
            assert plan.startswith("slice ") and " x_ahead=2" in plan and " waves=16 " in plan, plan
            X = synth.activations(M, K, 80 + M)
            X[M - 1, K - 1] = 3  # the last channel counts
            check(ams.ams_linear(packed, dev(scales), dev(X), N, fmt), O.linear(codes[rows], scales[rows], X, ofmt), rows, f"{ofmt.name} N={N} K={K} M={M}: {plan}")
