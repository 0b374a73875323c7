"""The quantizer where codes are looked up by magnitude (192 weights per scale and more) against the
oracle: rows just below and above that length, magnitudes drawn up to the row's largest and every one within
three units of a step of the code, subnormal weights, the smallest and largest scales; one scale per row, per
matrix and per run.  Codes and scales bit for bit."""

import numpy as np
import pytest

import paper_2510_16045_amd as ams
from oracle import ams_oracle as O

PAIRS = [(ams.FP533, O.FP533), (ams.FP425, O.FP425), (ams.FP45, O.FP45), (ams.FP433, O.FP433), (ams.FP6, O.FP6_E2M3), (ams.FP5, O.FP5_E2M2), (ams.FP4, O.FP4_E2M1)]


def rows(K, seed):
    rng = np.random.default_rng(seed)
    out = []
    for top in (0x0003, 0x0200, 0x0955, 0x2A66, 0x3C00, 0x51AB, 0x7BFF):  # largest magnitude of the row, as bits
        w = rng.integers(0, top + 1, size=K, dtype=np.uint16)  # uniform in bits: dense where the steps lie close
        w[K // 2] = top
        w |= (rng.integers(0, 2, size=K, dtype=np.uint16)) << 15
        out.append(w)
    return np.stack(out).view(np.float16)


@pytest.mark.parametrize("fmt,ofmt", PAIRS)
@pytest.mark.parametrize("search", ["set_bit", "reround"])
@pytest.mark.parametrize("K", [191, 192, 193, 512, 1537])
def test_codes_by_magnitude(fmt, ofmt, search, K):
    W = rows(K, K + fmt)
    packed, scales, codes = ams.ams_pack_ex(fmt, ams.SEARCH_REROUND if search == "reround" else ams.SEARCH_SET_BIT, W, return_codes=True)
    want, want_scales, _ = O.ams_quantize(W, ofmt, search="reround") if search == "reround" else O.ams_quantize(W, ofmt)
    assert np.array_equal(scales.view(np.uint16), want_scales.view(np.uint16))
    assert np.array_equal(codes, want)
    assert np.array_equal(ams.ams_unpack_host(fmt, packed, *W.shape), codes)


def around_the_steps(ofmt, top):
    """One row: the magnitudes (binary16 bits) within three of every midpoint and every value of the code at the row's
    own scale, both signs, the largest among them."""
    w = np.array([top], dtype=np.uint16).view(np.float16)
    s = float(O.ams_quantize(np.repeat(w, 2)[None, :], ofmt)[1][0])
    grid = O.magnitude_table(ofmt).astype(np.float64) * s
    marks = np.minimum(np.concatenate([grid, (grid[1:] + grid[:-1]) / 2]), 65504)
    bits = np.abs(marks).astype(np.float16).view(np.uint16).astype(np.int64)
    bits = np.unique(np.clip((bits[:, None] + np.arange(-3, 4)[None, :]).ravel(), 0, top))
    row = np.concatenate([[top], bits, bits | 0x8000]).astype(np.uint16)
    return np.random.default_rng(top).permutation(np.resize(row, max(row.size, 200))).view(np.float16)[None, :]


@pytest.mark.parametrize("fmt,ofmt", PAIRS)
@pytest.mark.parametrize("top", [0x0011, 0x0401, 0x2A66, 0x3C00, 0x7BFF])
def test_every_magnitude_around_the_steps(fmt, ofmt, top):
    W = around_the_steps(ofmt, top)
    for search in ("set_bit", "reround"):
        _, scales, codes = ams.ams_pack_ex(fmt, ams.SEARCH_REROUND if search == "reround" else ams.SEARCH_SET_BIT, W, return_codes=True)
        want, want_scales, _ = O.ams_quantize(W, ofmt, search="reround") if search == "reround" else O.ams_quantize(W, ofmt)
        assert np.array_equal(scales.view(np.uint16), want_scales.view(np.uint16))
        assert np.array_equal(codes, want)


@pytest.mark.parametrize("fmt,ofmt", PAIRS)
def test_other_granularities_look_up_too(fmt, ofmt):
    rec = 96 if ofmt.code_bits == 6 or fmt == ams.FP433 else 128
    W = rows(4 * rec + 201, 7 + fmt)
    _, scales, codes = ams.ams_pack_grouped(fmt, W, 2 * rec, return_codes=True)  # runs of 192 / 256, the last one of 201
    want, want_scales = O.ams_quantize_grouped(W, ofmt, 2 * rec)[:2]
    assert np.array_equal(codes, want)
    assert np.array_equal(scales[0].T[: W.shape[0]].view(np.uint16), np.asarray(want_scales).view(np.uint16))
    _, scales, codes = ams.ams_pack_per_tensor(fmt, W, return_codes=True)  # rows whose largest is not the matrix's
    want, want_scales, _ = O.ams_quantize(W, ofmt, per_tensor=True)
    assert np.array_equal(codes, want)
    assert np.array_equal(scales.view(np.uint16), want_scales.view(np.uint16))
