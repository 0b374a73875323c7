"""The quantizer where codes are looked up by magnitude (192 weights per scale and more) against the
oracle: rows just below and above that length, every magnitude up to the row's largest around the steps of
the code, subnormal weights, and the smallest and largest scales.  Codes and scales bit for bit."""

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
