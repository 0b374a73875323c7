"""The packer's vector paths: quantizing and packing in one pass (nobody asks for the codes) leaves the same bytes as
packing the codes that the oracle finds, at the edges of vectors, lane chunks, records and strips, for every scale
granularity; rows that make the first decision of a code or last bit unsure are decided exactly."""

import ctypes

import numpy as np
import pytest

import paper_2510_16045_amd as ams
from oracle import ams_oracle as O

PAIRS = [(ams.FP533, O.FP533), (ams.FP425, O.FP425), (ams.FP45, O.FP45), (ams.FP433, O.FP433), (ams.FP6, O.FP6_E2M3), (ams.FP5, O.FP5_E2M2), (ams.FP4, O.FP4_E2M1)]


def weights(N, K, seed):
    rng = np.random.default_rng(seed)
    W = (rng.standard_normal((N, K)) * np.exp2(rng.uniform(-18, 10, (N, 1)))).clip(-60000, 60000).astype(np.float16)
    W[0] = 0
    if K > 3:
        W[-1, 1], W[-1, 2] = -0.0, 6e-8
    return W


@pytest.mark.parametrize("fmt,ofmt", PAIRS)
@pytest.mark.parametrize("N,K", [(1, 1), (5, 23), (16, 24), (17, 32), (3, 47), (15, 48), (33, 63), (2, 64), (16, 95), (7, 96), (18, 97), (31, 128), (9, 129), (16, 511), (5, 515), (20, 1000)])
def test_one_pass_leaves_the_codes_bytes(fmt, ofmt, N, K):
    W = weights(N, K, 10 * K + fmt)
    codes, scales, _ = O.ams_quantize(W, ofmt)
    packed, got = ams.ams_pack(fmt, W)
    assert np.array_equal(got.view(np.uint16), scales.view(np.uint16))
    assert np.array_equal(packed, ams.ams_pack_codes(fmt, codes.astype(np.uint8)))
    again, _, with_codes = ams.ams_pack(fmt, W, return_codes=True)
    assert np.array_equal(with_codes, codes) and np.array_equal(again, packed)


@pytest.mark.parametrize("fmt,ofmt", PAIRS)
@pytest.mark.parametrize("runs", [1, 2, 3])
def test_one_pass_with_other_scales(fmt, ofmt, runs):
    rec = 96 if ofmt.code_bits == 6 or fmt == ams.FP433 else 128
    W = weights(19, rec * 4 * runs - 8, runs)
    packed, scales = ams.ams_pack_grouped(fmt, W, rec * 2)
    codes, want = O.ams_quantize_grouped(W, ofmt, rec * 2)[:2]
    assert np.array_equal(packed, ams.ams_pack_codes(fmt, codes.astype(np.uint8)))
    rows = scales.transpose(0, 2, 1).reshape(-1, scales.shape[1])
    assert np.array_equal(rows[:19].view(np.uint16), np.asarray(want).view(np.uint16)) and np.all(rows[19:] == 1)
    packed, _ = ams.ams_pack_per_tensor(fmt, W)
    codes = O.ams_quantize(W, ofmt, per_tensor=True)[0]
    assert np.array_equal(packed, ams.ams_pack_codes(fmt, codes.astype(np.uint8)))


@pytest.mark.parametrize("fmt,ofmt", PAIRS)
def test_ties_of_codes_and_of_errors(fmt, ofmt):
    # scale 1 and powers of two: the weights are multiples of a quarter of the smallest step, so that half of them lie on a tie
    # of two codes and many groups' squared errors are equal; and scales among the smallest binary16 numbers
    rng, fmax = np.random.default_rng(fmt), float(np.max(O.magnitude_table(ofmt)))
    rows = []
    for e in (-10, 0, 5):
        w = rng.integers(-int(fmax * 32), int(fmax * 32) + 1, 700) / 32.0 * 2.0**e
        w[0] = fmax * 2.0**e
        rows.append(w)
    for top in (1, 3, 11, 40):
        rows.append(rng.integers(-top, top + 1, 700) * 2.0**-24)
    W = np.stack(rows).astype(np.float16)
    codes, _, _ = O.ams_quantize(W, ofmt)
    assert np.array_equal(ams.ams_pack(fmt, W)[0], ams.ams_pack_codes(fmt, codes.astype(np.uint8)))
    for bad in (np.inf, -np.inf, np.nan):
        W[2, 699] = bad
        with pytest.raises(ams.AmsError):
            ams.ams_pack(fmt, W)


@pytest.mark.parametrize("fmt,ofmt", PAIRS)
@pytest.mark.parametrize("scale_group", [0, 1, 2])
@pytest.mark.parametrize("N,K,bad", [(3, 70, ((1, 69),)), (17, 300, ((0, 5), (16, 299))), (20, 1000, ((4, 999), (5, 400), (5, 600), (18, 0)))])
def test_rows_with_infinities_are_zero_codes(fmt, ofmt, scale_group, N, K, bad):
    # refused, with every byte of the matrix written all the same: the row or run with an inf or NaN as zero codes, its scale
    # left alone, and the others as ever, whether anybody asks for the codes (made first then) or not (one pass)
    rec = 96 if ofmt.code_bits == 6 or fmt == ams.FP433 else 128
    W = weights(N, K, K + fmt)
    lib, out = ams.load_library(), []
    codes = (O.ams_quantize_grouped(W, ofmt, rec * scale_group) if scale_group else O.ams_quantize(W, ofmt))[0]
    want = codes.astype(np.uint8)
    run = rec * scale_group or K
    for i, (n, k) in enumerate(bad):
        W[n, k] = (np.inf, -np.inf, np.nan)[i % 3]
        want[n, k // run * run : (k // run + 1) * run] = 0
    for codes_out in (None, np.empty((N, K), np.uint8)):
        packed = np.full(ams.ams_packed_bytes(fmt, N, K), 0xA5, np.uint8)
        got = np.full((N + 15) // 16 * 16 * -(-K // run), 0x1234, np.uint16)
        ptr = codes_out.ctypes.data if codes_out is not None else None
        if scale_group:
            rc = lib.ams_pack_grouped(fmt, 0, run, W.ctypes.data, N, K, K, packed.ctypes.data, got.ctypes.data, ptr)
        else:
            rc = lib.ams_pack_ex(fmt, 0, W.ctypes.data, N, K, K, packed.ctypes.data, got.ctypes.data, ptr)
        assert rc == -5  # AMS_ERR_NONFINITE
        assert np.array_equal(packed, ams.ams_pack_codes(fmt, want))
        out.append(got)
    assert np.array_equal(*out) and np.count_nonzero(out[0] == 0x1234) >= len({(n, k // run) for n, k in bad})


@pytest.mark.parametrize("fmt,ofmt", PAIRS)
@pytest.mark.parametrize("K", [5, 150, 700])  # candidates found one by one, and by intervals
def test_ties_of_the_rerounding_search(fmt, ofmt, K):
    # multiples of a quarter of the smallest step: midpoints between neighbouring candidates
    rng, fmax = np.random.default_rng(fmt + K), float(np.max(O.magnitude_table(ofmt)))
    W = (rng.integers(-int(fmax * 32), int(fmax * 32) + 1, (6, K)) / 32.0 * 2.0 ** rng.integers(-10, 6, (6, 1))).astype(np.float16)
    W[1:4, 0] = fmax * np.array([0.25, 1, 4])
    codes, scales, _ = O.ams_quantize(W, ofmt, search="reround")
    packed, got = ams.ams_pack_ex(fmt, ams.SEARCH_REROUND, W)
    assert np.array_equal(got.view(np.uint16), scales.view(np.uint16)) and np.array_equal(packed, ams.ams_pack_codes(fmt, codes.astype(np.uint8)))


def pack_lanes(lanes, fmt, W, scale_group, codes_out=False):
    """ams_pack* as a processor with vectors of `lanes` groups runs it; skips where this one has none so long."""
    N, K = W.shape
    fn = ams.load_library().ams_pack_lanes
    fn.argtypes = [ctypes.c_int] * 3 + [ctypes.c_int64, ctypes.c_void_p] + [ctypes.c_int64] * 3 + [ctypes.c_void_p] * 3
    packed = np.full(ams.ams_packed_bytes(fmt, N, K), 0xA5, np.uint8)
    n_scales = -(-N // 16) * 16 * -(-K // scale_group) if scale_group > 0 else N
    scales, codes = np.zeros(n_scales, np.float16), np.full((N, K), 0xA5, np.uint8)
    rc = fn(lanes, fmt, ams.SEARCH_SET_BIT, scale_group, W.ctypes.data, N, K, K, packed.ctypes.data, scales.ctypes.data, codes.ctypes.data if codes_out else None)
    if rc == -7:  # AMS_ERR_DEVICE
        pytest.skip(f"no vectors of {lanes} groups on this processor")
    assert rc == 0
    return packed, scales, codes


def tied_weights(fmt, ofmt, K):
    rng, fmax = np.random.default_rng(fmt), float(np.max(O.magnitude_table(ofmt)))
    rows = [rng.integers(-int(fmax * 32), int(fmax * 32) + 1, K) / 32.0 * 2.0**e for e in (-10, 0, 5)]
    for w, e in zip(rows, (-10, 0, 5)):
        w[0] = fmax * 2.0**e
    return np.stack(rows + [rng.integers(-top, top + 1, K) * 2.0**-24 for top in (1, 3, 11, 40)]).astype(np.float16)


@pytest.mark.parametrize("lanes", [16, 8, 0])
@pytest.mark.parametrize("fmt,ofmt", PAIRS)
def test_every_vector_length_leaves_the_codes_bytes(fmt, ofmt, lanes):
    # every instruction set's path, whatever this processor would take: with 16 groups at a time, with 8, looked up
    rec = 96 if ofmt.code_bits == 6 or fmt == ams.FP433 else 128
    for N, K in ((1, 1), (5, 23), (16, 24), (17, 32), (3, 47), (15, 48), (33, 63), (2, 64), (7, 96), (18, 97), (31, 128), (9, 129), (16, 511), (5, 515), (20, 1000), (7, 700)):
        W = tied_weights(fmt, ofmt, K) if K == 700 else weights(N, K, 10 * K + fmt)
        codes, scales, _ = O.ams_quantize(W, ofmt)
        want = ams.ams_pack_codes(fmt, codes.astype(np.uint8))
        for codes_out in (False, True):
            packed, got, out = pack_lanes(lanes, fmt, W, 0, codes_out)
            assert np.array_equal(packed, want) and np.array_equal(got.view(np.uint16), scales.view(np.uint16)), (N, K)
            assert not codes_out or np.array_equal(out, codes), (N, K)
        packed, _, _ = pack_lanes(lanes, fmt, W, -1)
        assert np.array_equal(packed, ams.ams_pack_codes(fmt, O.ams_quantize(W, ofmt, per_tensor=True)[0].astype(np.uint8))), (N, K)
        packed, _, _ = pack_lanes(lanes, fmt, W, 2 * rec)
        assert np.array_equal(packed, ams.ams_pack_codes(fmt, O.ams_quantize_grouped(W, ofmt, 2 * rec)[0].astype(np.uint8))), (N, K)
