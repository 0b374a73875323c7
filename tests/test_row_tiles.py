"""The rows of X dealt to several workgroups (slice plans with row_tiles): where the plan does it, and the results
at uneven tiles, ragged strips, grids that are not whole groups of eight, scales per run and a split K."""

import numpy as np
import pytest

import paper_2510_16045_amd as ams
from oracle import ams_oracle as O
from paper_2510_16045_amd import synth
from test_gpu_slice_kernel import PAIRS, REC_K, check, dev, problem, scales_per_run

torch = pytest.importorskip("torch")


def plan(*a, **k):
    text = ams.ams_linear_plan(*a, **k).split()
    return text[0], dict(kv.split("=") for kv in text[1:])


@pytest.mark.parametrize(
    "fmt,M,N,K,entry,tiles",
    [
        (ams.FP425, 32, 4096, 14336, 0, 2), (ams.FP425, 16, 4096, 14336, 0, 2), (ams.FP425, 15, 4096, 14336, 0, 1), (ams.FP425, 32, 28672, 4096, 0, 1),
        (ams.FP533, 24, 2560, 9728, 0, 3), (ams.FP533, 32, 1024, 4096, 0, 4), (ams.FP533, 16, 8192, 8192, 0, 1), (ams.FP533, 32, 8192, 8192, 0, 2),
        (ams.FP533, 32, 4096, 17 * 96, 0, 1), (ams.FP533, 32, 4096, 18 * 96, 0, 2), (ams.FP533, 32, 28672, 4099, 0, 1),  # too few records; unaligned rows on too many strips
        (ams.FP533, 16, 4608, 2368, 2, 1), (ams.FP533, 16, 4608, 2368, 0, 2),  # scales per run
        (ams.FP425, 32, 2560, 9728, 1, 2),
        (ams.FP6, 16, 2739, 1920, 0, 1), (ams.FP6, 16, 2048, 1920, 0, 2), (ams.FP6, 17, 2739, 1920, 0, 2), (ams.FP45, 16, 2739, 1920 * 2, 0, 2),  # 16 rows, a second strip
        (ams.FP433, 16, 2155, 2776, 2, 1), (ams.FP433, 16, 2155, 96 * 96, 2, 1), (ams.FP433, 16, 2155, 97 * 96, 2, 2), (ams.FP433, 16, 2155, 32 * 96, 0, 1), (ams.FP433, 16, 2155, 33 * 96, 0, 2),
    ],
)
def test_where_the_rows_are_dealt(fmt, M, N, K, entry, tiles):
    kind, p = plan(fmt, M, N, K, with_workspace=entry)
    assert int(p.get("row_tiles", 1)) == tiles, p
    if tiles > 1:
        assert kind == "slice" and int(p["rows_per_tile"]) == -(-M // tiles), p


def test_every_plan_covers_the_matrix_in_one_round():
    rng = np.random.default_rng(5)
    seen = set()
    for _ in range(20000):
        fmt, M = int(rng.integers(7)), int(rng.integers(16, 33))
        N, K, entry = int(2 ** rng.uniform(4, 15)), int(2 ** rng.uniform(10, 15)) // 8 * 8, int(rng.integers(3))
        kind, p = plan(fmt, M, N, K, with_workspace=entry)
        if "row_tiles" not in p:
            continue
        tiles, grid, spw, slices = (int(p[k]) for k in ("row_tiles", "grid", "strips_per_wg", "k_slices"))
        seen.add((tiles, slices > 1))
        assert grid <= 256 and grid % (8 * tiles) == 0 and 1 <= spw <= 8, (fmt, M, N, K, p)
        assert grid // tiles >= -(-(-(-N // 16)) // spw) * slices, (fmt, M, N, K, p)
        assert int(p["rows_per_tile"]) * tiles >= M > int(p["rows_per_tile"]) * (tiles - 1), (fmt, M, N, K, p)
        assert int(p["lds"]) <= 160 * 1024
    assert {(2, False), (3, False), (4, False), (2, True)} <= seen, seen


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,ofmt", PAIRS)
@pytest.mark.parametrize("N,n_rec,Ms", [(4091, 19, (16, 17, 32)), (2555, 34, (24, 25, 31)), (200, 40, (32, 27)), (6139, 18, (29,))])
def test_row_tiles(fmt, ofmt, N, n_rec, Ms):
    K = REC_K[fmt] * n_rec - 8 * (n_rec % 3)
    codes, scales, rows = problem(fmt, ofmt, N, K, N + n_rec)
    wp, sc = dev(ams.ams_pack_codes(fmt, codes)), dev(scales)
    for M in Ms:
        kind, p = plan(fmt, M, N, K)
        assert (int(p.get("row_tiles", 1)) > 1) == (M > 16 or fmt not in (ams.FP433, ams.FP6)), p  # 16 rows: a second strip costs those two too much
        X = synth.activations(M, K, 40 + M)
        ref = O.linear(codes[rows], scales[rows], X, ofmt)
        x, what = dev(X), f"{ofmt.name} N={N} K={K} M={M}: {p}"
        guard = torch.full((M + 2, N), 7.0, dtype=torch.float16, device="cuda")  # rows before and behind Y stay as they are
        if N % 8 == 0:
            ams.ams_linear(wp, sc, x, N, fmt, out=guard[1 : M + 1])
            check(guard[1 : M + 1], ref, rows, what)
            assert torch.all(guard[0] == 7) and torch.all(guard[M + 1] == 7), what
        else:
            check(ams.ams_linear(wp, sc, x, N, fmt), ref, rows, what)
        x[M // 2] = float("inf")
        check(ams.ams_linear(wp, sc, x, N, fmt), ref, rows, "beside a row of infinities: " + what, [m for m in range(M) if m != M // 2])


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,ofmt", PAIRS)
def test_row_tiles_with_one_scale_per_run(fmt, ofmt):
    N, M, n_rec = 4091, 31, 21
    K, sg = REC_K[fmt] * n_rec - 16, 2 * REC_K[fmt]
    kind, p = plan(fmt, M, N, K, with_workspace=2)
    assert int(p.get("row_tiles", 1)) > 1, p
    codes, _, rows = problem(fmt, ofmt, N, K, 12)
    scales, packed = scales_per_run(N, K, sg, 3)
    X = synth.activations(M, K, 41)
    y = ams.ams_linear_grouped(dev(ams.ams_pack_codes(fmt, codes)), dev(packed), sg, dev(X), N, fmt)
    check(y, O.linear(codes[rows], scales[rows], X, ofmt, sg), rows, f"{ofmt.name}: {p}")


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,ofmt", PAIRS)
@pytest.mark.parametrize("N,K,M", [(2555, 9728, 32), (1275, 9736, 32)])
def test_row_tiles_and_slices_of_k(fmt, ofmt, N, K, M):
    kind, p = plan(fmt, M, N, K, with_workspace=True)
    assert int(p.get("row_tiles", 1)) > 1 and int(p["k_slices"]) > 1, p
    codes, scales, rows = problem(fmt, ofmt, N, K, 8)
    wp, sc, X = dev(ams.ams_pack_codes(fmt, codes)), dev(scales), synth.activations(M, K, 42)
    ws = torch.zeros(16 << 20, dtype=torch.uint8, device="cuda")
    x, what = dev(X), f"{ofmt.name} N={N} K={K} M={M}: {p}"
    first = ams.ams_linear_ws(wp, sc, x, N, fmt, ws)
    check(first, O.linear(codes[rows], scales[rows], X, ofmt), rows, what)
    for _ in range(3):
        assert torch.equal(ams.ams_linear_ws(wp, sc, x, N, fmt, ws), first), what
    assert torch.equal(ams.ams_linear_static_ws(wp, sc, x, N, fmt), first), what
    assert not ws[: 4 * 16384].any(), what
