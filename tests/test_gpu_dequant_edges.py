"""ams_dequant where its row-wise stores can go wrong: rows shorter than one 16-byte store, rows that
end inside one, rows and buffers that start anywhere, ragged strips, and scales whose products are
subnormal or overflow.  Bit for bit against the oracle, and nothing outside the matrix is touched."""

import numpy as np
import pytest

import paper_2510_16045_amd as ams
from oracle import ams_oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

PAIRS = [(ams.FP533, O.FP533), (ams.FP425, O.FP425), (ams.FP45, O.FP45), (ams.FP433, O.FP433), (ams.FP6, O.FP6_E2M3), (ams.FP5, O.FP5_E2M2), (ams.FP4, O.FP4_E2M1)]


@pytest.mark.parametrize("fmt,ofmt", PAIRS)
@pytest.mark.parametrize("N,K", [(1, 1), (16, 7), (17, 8), (15, 9), (33, 95), (18, 97), (5, 128), (31, 130), (16, 513), (64, 1031)])
def test_dequant_edges(fmt, ofmt, N, K):
    rng = np.random.default_rng(1000 * N + K)
    codes = rng.integers(0, 1 << ofmt.code_bits, size=(N, K), dtype=np.uint8)
    last = np.repeat(codes[:, :: ofmt.group] & 1, ofmt.group, axis=1)[:, :K]
    codes = (codes & 0xFE) | last
    s = np.exp2(rng.uniform(-24, 16, size=N)).astype(np.float16)  # products from below the smallest subnormal to infinity
    s[s == np.inf] = np.float16(65504)
    wp = torch.from_numpy(ams.ams_pack_codes(fmt, codes)).cuda()
    sc = torch.from_numpy(s.view(np.int16)).cuda().view(torch.float16)
    with np.errstate(over="ignore"):
        want = O.dequant_scaled(codes, s, ofmt).view(np.uint16)
    for shift in (0, 1, 3, 8):  # halfs by which the result starts behind a 16-byte boundary
        whole = torch.full((N * K + 16,), 7.0, dtype=torch.float16, device="cuda")
        out = whole[shift : shift + N * K].view(N, K)
        ams.ams_dequant(fmt, wp, sc, N, K, scaled=True, out=out)
        got = whole.cpu().view(torch.int16).numpy().view(np.uint16)
        assert np.array_equal(got[shift : shift + N * K].reshape(N, K), want), f"shift {shift}"
        outside = np.r_[got[:shift], got[shift + N * K :]]
        assert np.all(outside == np.float16(7.0).view(np.uint16)), f"shift {shift}: stored outside"
