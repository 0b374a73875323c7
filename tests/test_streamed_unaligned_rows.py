"""slice_kernel's variant for activation rows that are not 16-byte aligned (plans with streamed_rows): every number of
strips and of row tiles, wavefronts with no, one and many records, every remainder of K, ragged strips, K split over
workgroups; sampled rows against the oracle.  One activation row of infinities must leave the others alone."""

import numpy as np
import pytest

import paper_2510_16045_amd as ams
from oracle import ams_oracle as O
from paper_2510_16045_amd import synth
from test_gpu_slice_kernel import PAIRS, REC_K, check, dev, problem

torch = pytest.importorskip("torch")


def plan(*a, **k):
    text = ams.ams_linear_plan(*a, **k).split()
    return text[0], dict(kv.split("=") for kv in text[1:])


@pytest.mark.parametrize(
    "fmt,M,N,K,entry,tiles",
    [
        (ams.FP533, 5, 11003, 4099, 0, 1), (ams.FP425, 8, 4096, 4099, 0, 1), (ams.FP425, 9, 4096, 4099, 0, 2), (ams.FP425, 32, 4096, 14337, 0, 4),
        (ams.FP425, 32, 4112, 14337, 0, 0), (ams.FP425, 16, 8192, 4099, 0, 2), (ams.FP425, 16, 8208, 4099, 0, 0), (ams.FP425, 4, 16384, 4099, 0, 1), (ams.FP425, 4, 16400, 4099, 0, 0),
        (ams.FP425, 8, 4096, 14339, 0, 1), (ams.FP425, 8, 4112, 14339, 0, 1), (ams.FP425, 8, 200, 14339, 0, 1), (ams.FP425, 7, 4096, 14339, 0, 1), (ams.FP425, 4, 256, 129, 0, 1), (ams.FP425, 4, 256, 127, 0, 0), (ams.FP533, 4, 256, 97, 2, 0),
        (ams.FP533, 1, 8192, 8193, 0, 0), (ams.FP533, 3, 8192, 8193, 0, 1),
        (ams.FP45, 1, 355, 24567, 0, 0), (ams.FP425, 1, 355, 28159, 0, 1), (ams.FP425, 1, 355, 28161, 0, 0), (ams.FP533, 1, 355, 105783, 0, 0), (ams.FP533, 2, 355, 105783, 0, 1),  # long K
        (ams.FP533, 12, 6285, 2727, 0, 0), (ams.FP533, 12, 6285, 2687, 0, 2), (ams.FP533, 12, 6140, 2727, 0, 2), (ams.FP533, 12, 6285, 4099, 0, 2),  # two tiles of four strips
        (ams.FP533, 13, 6285, 3071, 0, 0), (ams.FP533, 13, 6285, 3073, 0, 2), (ams.FP6, 15, 6552, 2857, 0, 0), (ams.FP533, 12, 6285, 5999, 0, 0), (ams.FP533, 13, 6285, 5999, 0, 2),
        (ams.FP425, 9, 6285, 4099, 0, 0), (ams.FP425, 10, 6285, 4099, 0, 2), (ams.FP5, 10, 6285, 4099, 0, 0), (ams.FP5, 11, 6285, 4099, 0, 2), (ams.FP6, 12, 6285, 29179, 0, 0), (ams.FP6, 13, 6285, 29179, 0, 2),
    ],
)
def test_where_unaligned_rows_are_streamed(fmt, M, N, K, entry, tiles):
    kind, p = plan(fmt, M, N, K, with_workspace=entry)
    assert kind == ("slice" if tiles else "column") and int(p.get("row_tiles", 0)) == tiles and ("streamed_rows" in p) == (tiles > 0), p
    if tiles:
        assert int(p["streamed_rows"]) == -(-M // tiles) <= 8 and p["waves"] == "16" and int(p["strips_per_wg"]) <= 4
        assert int(p["grid"]) // tiles * int(p["strips_per_wg"]) >= -(-N // 16) * int(p["k_slices"]) and int(p["grid"]) <= 256


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,ofmt", PAIRS)
@pytest.mark.parametrize("spw", [1, 2, 3, 4])
def test_strips_records_and_remainders(fmt, ofmt, spw):
    N = 16 * (256 * (spw - 1) + 130) - 5 if spw > 1 else 16 * 130 - 5
    for n_rec, rest, Ms in ((2, 1, (1, 8)), (3, 7, (3,)), (17, 2, (4, 7)), (18, 3, (2, 8)), (33, 4, (5,)), (34, 5, (1, 6)), (50, 6, (4,))):
        K = REC_K[fmt] * (n_rec - 1) + 8 * (n_rec % 4) + rest
        codes, scales, rows = problem(fmt, ofmt, N, K, 100 * spw + n_rec)
        wp, sc = dev(ams.ams_pack_codes(fmt, codes)), dev(scales)
        for M in Ms:
            _, p = plan(fmt, M, N, K)
            if "streamed_rows" not in p:  # three records ahead in column_kernel: formats without side groups at M <= 2
                assert p["ahead"] == "3", p
                continue
            assert int(p["strips_per_wg"]) == spw, p
            X = synth.activations(M, K, 30 + M)
            ref = O.linear(codes[rows], scales[rows], X, ofmt)
            x, what = dev(X), f"{ofmt.name} N={N} K={K} M={M}: {p}"
            check(ams.ams_linear(wp, sc, x, N, fmt), ref, rows, what)
            if M > 2:
                x[M // 2] = float("inf")
                check(ams.ams_linear(wp, sc, x, N, fmt), ref, rows, "beside a row of infinities: " + what, [m for m in range(M) if m != M // 2])


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,ofmt", PAIRS)
@pytest.mark.parametrize("N,K,M,entry", [(4091, 2051, 9, "plain"), (2555, 4099, 24, "plain"), (600, 1501, 32, "plain"), (4000, 1001, 17, "plain"), (700, 12803, 15, "ws"), (1003, 9731, 31, "ws"), (1003, 9731, 6, "ws")])
def test_row_tiles_and_slices_of_k(fmt, ofmt, N, K, M, entry):
    _, p = plan(fmt, M, N, K, with_workspace=entry == "ws")
    assert int(p.get("row_tiles", 0)) == -(-M // 8), p
    codes, scales, rows = problem(fmt, ofmt, N, K, 8)
    wp, sc, X = dev(ams.ams_pack_codes(fmt, codes)), dev(scales), synth.activations(M, K, 42)
    ws = torch.zeros(16 << 20, dtype=torch.uint8, device="cuda")
    x, what = dev(X), f"{ofmt.name} N={N} K={K} M={M}: {p}"
    call = lambda: ams.ams_linear_ws(wp, sc, x, N, fmt, ws) if entry == "ws" else ams.ams_linear(wp, sc, x, N, fmt)
    first, ref = call(), O.linear(codes[rows], scales[rows], X, ofmt)
    check(first, ref, rows, what)
    for _ in range(3):
        assert torch.equal(call(), first), what
    assert not ws[: 4 * 16384].any(), what
    x[M // 2] = float("inf")
    check(call(), ref, rows, "beside a row of infinities: " + what, [m for m in range(M) if m != M // 2])
