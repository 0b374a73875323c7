"""The Linear on activation rows that are not 16-byte aligned (K % 8 != 0): every remainder, rows shorter
than one 16-byte load, and every launch variant (side groups dealt whole, three records ahead, two strips
per wavefront, several phases of K, one scale per run).  Rows must not see each other: one row of
infinities leaves the others' results alone."""

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


def check(y, ref, rows, what):
    # fp32 sums rounded to fp16: 2^-11 relative per output at most, half of it in the mean; 1e-3 as everywhere
    y = y.cpu().view(torch.int16).numpy().view(np.float16).astype(np.float64)[rows]
    assert np.all(np.isfinite(y)), what
    assert np.linalg.norm(y - ref[rows]) <= 1e-3 * np.linalg.norm(ref[rows]), what


@pytest.mark.parametrize("fmt,ofmt", PAIRS)
@pytest.mark.parametrize("K", [1, 7, 9, 10, 95, 97, 259, 516, 773, 1030, 1287, 2052 + 1, 4099])
def test_every_remainder(fmt, ofmt, K):
    N = 40
    W = synth.gaussian_weights(N, K, 60)
    packed, scales = ams.ams_pack(fmt, W)
    codes, o_scales, _ = O.ams_quantize(W, ofmt)
    gp, gs = ams.ams_pack_grouped(fmt, W, REC_K[fmt])
    g_codes, g_scales = O.ams_quantize_grouped(W, ofmt, REC_K[fmt])
    for M in (1, 5, 16, 32):
        X = synth.activations(M, K, 61 + M)
        ref, g_ref = O.linear(codes, o_scales, X, ofmt), O.linear(g_codes, g_scales, X, ofmt, REC_K[fmt])
        x = dev(X)
        check(ams.ams_linear(dev(packed), dev(scales), x, N, fmt), ref, slice(None), f"{ofmt.name} K={K} M={M}")
        check(ams.ams_linear_grouped(dev(gp), dev(gs), REC_K[fmt], x, N, fmt), g_ref, slice(None), f"{ofmt.name} K={K} M={M} grouped")
        if M > 1:
            bad = M // 2
            x[bad] = float("inf")
            rest = [m for m in range(M) if m != bad]
            check(ams.ams_linear(dev(packed), dev(scales), x, N, fmt), ref, rest, f"{ofmt.name} K={K} M={M}: beside a row of infinities")


@pytest.mark.parametrize(
    "fmt,ofmt,N,K,M,want",
    [
        (ams.FP425, O.FP425, 16 * 7 * 230, 2051, 2, "waves=8 waves_per_strip=1 "),  # three records ahead in the side-group deal
        (ams.FP533, O.FP533, 16 * 7 * 230, 2051, 2, "ahead=3"),
        (ams.FP533, O.FP533, 16 * 11 * 230, 1003, 3, "strips_per_wave=2"),
        (ams.FP6, O.FP6_E2M3, 20496, 96 * 12 - 5, 5, "side_groups=1"),
        (ams.FP433, O.FP433, 20496, 96 * 24 - 3, 1, "side_groups=1"),
        (ams.FP45, O.FP45, 20500, 4501, 32, "phases=3 "),  # K in several phases
    ],
)
def test_every_launch_variant(fmt, ofmt, N, K, M, want):
    assert want in ams.ams_linear_plan(fmt, M, N, K)
    W = synth.gaussian_weights(N, K, 62)
    packed, scales = ams.ams_pack(fmt, W)
    rows = np.unique(np.r_[0:16, N - 16 : N, np.arange(7, N, 997)])
    codes, o_scales, _ = O.ams_quantize(W[rows], ofmt)
    X = synth.activations(M, K, 63)
    y = ams.ams_linear(dev(packed), dev(scales), dev(X), N, fmt)[:, torch.from_numpy(rows).cuda()].contiguous()
    check(y, O.linear(codes, o_scales, X, ofmt), slice(None), f"{ofmt.name} N={N} K={K} M={M}")


@pytest.mark.parametrize("fmt,ofmt,K", [(ams.FP533, O.FP533, 25601), (ams.FP425, O.FP425, 25603), (ams.FP6, O.FP6_E2M3, 25607)])
def test_slices_of_k_in_phases(fmt, ofmt, K):
    # more strips than the tiles of a split take: column_kernel, each of eight slices of K in two phases
    N, M = 600, 32
    plan = ams.ams_linear_plan(fmt, M, N, K, with_workspace=True)
    assert plan.startswith("column ") and "k_slices=8 " in plan and "phases=2 " in plan, plan
    W = synth.gaussian_weights(N, K, 64)
    packed, scales = ams.ams_pack(fmt, W)
    codes, o_scales, _ = O.ams_quantize(W, ofmt)
    X, ws = synth.activations(M, K, 65), torch.zeros(16 << 20, dtype=torch.uint8, device="cuda")
    wp, sc, x = dev(packed), dev(scales), dev(X)
    first, ref = ams.ams_linear_ws(wp, sc, x, N, fmt, ws), O.linear(codes, o_scales, X, ofmt)
    check(first, ref, slice(None), plan)
    assert torch.equal(ams.ams_linear_ws(wp, sc, x, N, fmt, ws), first) and torch.equal(ams.ams_linear_static_ws(wp, sc, x, N, fmt), first)
    assert not ws[: 4 * 16384].any()
