"""The rows of X dealt to workgroups that would have none otherwise: up to 128 strips, from five rows on, tiles of four rows and
more.  Where the plan does it, and the results at uneven tiles, ragged strips, scales per run and records from one on."""

import pytest

import paper_2510_16045_amd as ams
from oracle import ams_oracle as O
from paper_2510_16045_amd import synth
from test_gpu_slice_kernel import PAIRS, REC_K, check, dev, problem, scales_per_run

torch = pytest.importorskip("torch")


def tiles(*a, **k):
    kind, *kv = ams.ams_linear_plan(*a, **k).split()
    p = dict(x.split("=") for x in kv)
    assert kind == "slice" and p["strips_per_wg"] == "1", (a, p)
    return int(p.get("row_tiles", 1))


@pytest.mark.parametrize("fmt", range(7))
def test_where_the_rows_are_dealt(fmt):
    rec = REC_K[fmt]
    for strips, most in ((128, 2), (129, 1), (80, 3), (81, 2), (64, 4), (65, 3), (3, 4)):
        for M, want in ((4, 1), (5, 2), (8, 2), (9, 3), (12, 3), (13, 4), (16, 4), (17, 4), (32, 4)):
            assert tiles(fmt, M, 16 * strips - 5, 9 * rec) == min(want, most), (strips, M)
    for M, n_rec, strips, want in ((8, 1, 128, 2), (12, 8, 80, 3), (12, 8, 128, 1), (13, 8, 80, 1), (16, 8, 64, 4), (16, 9, 80, 3), (17, 1, 128, 2)):
        assert tiles(fmt, M, 16 * strips, n_rec * rec) == want, (M, n_rec, strips)
    assert tiles(fmt, 16, 1024, 40 * rec) == tiles(fmt, 16, 1024, 40 * rec, with_workspace=2) == 4  # by the cost of a step of K
    assert tiles(fmt, 16, 1280, 40 * rec) == 3


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,ofmt", PAIRS)
@pytest.mark.parametrize("N,n_rec,Ms", [(1003, 1, (5, 13, 17)), (1275, 9, (9, 11, 31)), (2043, 25, (6, 15, 18)), (37, 40, (7, 10, 14, 29))])
def test_results(fmt, ofmt, N, n_rec, Ms):
    K, sg = REC_K[fmt] * n_rec - 8 * (n_rec % 3), REC_K[fmt]
    codes, scales, rows = problem(fmt, ofmt, N, K, N + n_rec)
    run_scales, run_packed = scales_per_run(N, K, sg, 5)
    wp, sc, run_sc = dev(ams.ams_pack_codes(fmt, codes)), dev(scales), dev(run_packed)
    for M in Ms:
        n = tiles(fmt, M, N, K)
        assert n > 1 or (n_rec <= 8 and M <= 16)
        X = synth.activations(M, K, 40 + M)
        ref = O.linear(codes[rows], scales[rows], X, ofmt)
        x, what = dev(X), f"{ofmt.name} N={N} K={K} M={M}: {n} tiles"
        check(ams.ams_linear(wp, sc, x, N, fmt), ref, rows, what)
        check(ams.ams_linear_grouped(wp, run_sc, sg, x, N, fmt), O.linear(codes[rows], run_scales[rows], X, ofmt, sg), rows, "scales per run, " + what)
        x[M // 2] = float("inf")
        check(ams.ams_linear(wp, sc, x, N, fmt), ref, rows, "beside a row of infinities: " + what, [m for m in range(M) if m != M // 2])
