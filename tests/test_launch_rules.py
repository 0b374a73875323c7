"""Which kernel a Linear gets where the choice was measured to matter: shapes on which slice_kernel was the slower one
stay on column_kernel, and slice_kernel's workgroups keep the sizes that its rules assume.  Host only."""

import numpy as np
import pytest

import paper_2510_16045_amd as ams


def plan(*a, **k):
    text = ams.ams_linear_plan(*a, **k).split()
    return text[0], dict(kv.split("=") for kv in text[1:])


@pytest.mark.parametrize("M", [3, 4])
@pytest.mark.parametrize("N,K", [(48000, 128), (65536, 1536), (128256, 640)])
def test_two_workgroups_of_fp433_fit_on_a_compute_unit(M, N, K):
    # more than eight strips for every compute unit are dealt to two workgroups, which have to run side by side: with
    # sixteen wavefronts of 88 to 106 registers each they took turns
    kind, p = plan(ams.FP433, M, N, K)
    assert kind == "slice" and int(p["strips_per_wg"]) in (6, 8) and p["waves"] == "8", p


GROUPED = 2  # of the plan query's with_workspace


@pytest.mark.parametrize(
    "fmt,M,N,K,entry",
    [
        (ams.FP45, 4, 65536, 256, 0),  # an even number of records that is no multiple of four, two to a side group
        (ams.FP6, 3, 65536, 96 * 14, 0),
        (ams.FP6, 3, 128256, 96, 0),
        (ams.FP533, 3, 65536, 96, GROUPED),  # few records per wavefront
        (ams.FP433, 4, 65536, 96 * 15, GROUPED),
        (ams.FP533, 4, 128256, 192, GROUPED),
        (ams.FP425, 4, 65536, 128, GROUPED),  # workgroups that do not fit on a compute unit together
        (ams.FP425, 3, 128256, 28 * 128, GROUPED),
        (ams.FP5, 4, 65536, 63 * 128, GROUPED),
        (ams.FP4, 4, 65536, 63 * 128, GROUPED),
        (ams.FP425, 32, 45000, 79 * 128, 0),
        (ams.FP533, 24, 45000, 70 * 96, GROUPED),
        (ams.FP533, 16, 45000, 63 * 96, 0),
    ],
)
def test_more_than_eight_strips_where_one_workgroup_is_faster(fmt, M, N, K, entry):
    assert plan(fmt, M, N, K, with_workspace=entry)[0] == "column"


@pytest.mark.parametrize(
    "fmt,M,N,K,entry",
    [
        (ams.FP45, 4, 65536, 384, 0), (ams.FP45, 4, 65536, 26 * 128, 0), (ams.FP6, 3, 128256, 288, 0), (ams.FP425, 4, 65536, 128, 0),
        (ams.FP533, 3, 65536, 96 * 16, GROUPED), (ams.FP533, 3, 36000, 96 * 3, GROUPED), (ams.FP533, 4, 128256, 96 * 3, GROUPED),
        (ams.FP425, 4, 65536, 24 * 128, GROUPED), (ams.FP425, 3, 128256, 32 * 128, GROUPED), (ams.FP5, 4, 65536, 64 * 128, GROUPED),
        (ams.FP4, 4, 56000, 16 * 128, GROUPED), (ams.FP425, 32, 45000, 80 * 128, 0), (ams.FP425, 32, 128256, 64 * 128, 0),
        (ams.FP533, 16, 45000, 64 * 96, 0),
    ],
)
def test_more_than_eight_strips_where_two_workgroups_are_faster(fmt, M, N, K, entry):
    kind, p = plan(fmt, M, N, K, with_workspace=entry)
    strips = min(16, -(-(-(-N // 16)) // 256))
    assert kind == "slice" and int(p["strips_per_wg"]) == (strips + 1) // 2, p


@pytest.mark.parametrize("fmt", range(7))
@pytest.mark.parametrize(
    "M,strips,n_rec,entry,want",
    [
        (17, 8, 16, 0, "column"), (32, 8, 1, GROUPED, "column"), (32, 8, 17, 0, "slice"), (32, 8, 17, GROUPED, "slice"),
        (16, 8, 2, 0, "column"), (16, 8, 3, 0, "slice"), (8, 8, 1, 0, "slice"),
        (32, 7, 2, 0, "column"), (32, 7, 3, 0, "slice"), (32, 7, 43, 0, "slice"), (16, 7, 1, GROUPED, "slice"),
        (24, 6, 1, 0, "column"), (24, 6, 2, 0, "column"), (24, 6, 3, 0, "slice"), (24, 6, 2, GROUPED, "column"), (24, 6, 3, GROUPED, "slice"), (32, 5, 1, 0, "slice"),
    ],
)
def test_few_records_at_large_batches(fmt, M, strips, n_rec, entry, want):
    rec = 96 if fmt in (ams.FP533, ams.FP433, ams.FP6) else 128
    kind, p = plan(fmt, M, 16 * 256 * strips - 5, rec * n_rec, with_workspace=entry)
    assert kind == want and int(p["strips_per_wg"]) == strips, p


@pytest.mark.parametrize(
    "fmt,M,N,n_rec,entry,want",
    [
        (ams.FP425, 1, 6144, 97, 0, "column"), (ams.FP533, 1, 6144, 97, GROUPED, "column"), (ams.FP533, 1, 6144, 96, 0, "slice"),
        (ams.FP533, 1, 6144, 43, 0, "slice"), (ams.FP5, 1, 6144, 127, 0, "slice"), (ams.FP5, 1, 6144, 97, GROUPED, "column"), (ams.FP425, 2, 6144, 127, 0, "slice"), (ams.FP425, 2, 6144, 128, 0, "column"),
        (ams.FP425, 1, 8192, 128, 0, "slice"),  # every compute unit has two strips
        (ams.FP6, 1, 8192, 97, GROUPED, "column"), (ams.FP5, 1, 16384, 96, GROUPED, "slice"), (ams.FP5, 2, 16384, 145, GROUPED, "column"),
        (ams.FP45, 2, 8192, 200, GROUPED, "slice"), (ams.FP45, 2, 8192, 201, GROUPED, "column"), (ams.FP6, 2, 12288, 150, GROUPED, "slice"),
        (ams.FP533, 1, 16384, 201, GROUPED, "column"), (ams.FP533, 1, 16384, 200, GROUPED, "slice"), (ams.FP533, 1, 16384, 250, 0, "slice"),
        (ams.FP6, 1, 16384, 201, 0, "column"), (ams.FP433, 1, 1000, 201, 0, "column"), (ams.FP425, 1, 1000, 250, 0, "slice"),
        (ams.FP533, 1, 1000, 201, GROUPED, "column"), (ams.FP5, 1, 1000, 201, GROUPED, "slice"), (ams.FP4, 1, 16384, 250, GROUPED, "slice"),
        (ams.FP6, 2, 16384, 250, 0, "slice"), (ams.FP6, 3, 6144, 250, 0, "slice"),
    ],
)
def test_long_k_at_small_batches(fmt, M, N, n_rec, entry, want):
    rec = 96 if fmt in (ams.FP533, ams.FP433, ams.FP6) else 128
    assert plan(fmt, M, N, rec * n_rec, with_workspace=entry)[0] == want


@pytest.mark.parametrize(
    "fmt,M,N,K,slices,want",
    [
        (ams.FP533, 16, 2560, 18944, 8, "column"), (ams.FP533, 16, 2560, 25600, 8, "slice"), (ams.FP425, 16, 2560, 25600, 8, "slice"),
        (ams.FP6, 16, 3584, 22016, 8, "column"), (ams.FP425, 32, 2048, 25600, 8, "column"), (ams.FP425, 16, 1536, 13824, 8, "slice"),
        (ams.FP425, 32, 1536, 13824, 8, "column"), (ams.FP425, 32, 1536, 18944, 8, "slice"), (ams.FP533, 32, 1536, 18944, 8, "column"),
        (ams.FP533, 32, 5120, 9600, 4, "column"), (ams.FP433, 32, 5120, 11008, 4, "column"), (ams.FP425, 32, 5120, 11008, 4, "slice"),
        (ams.FP45, 32, 2048, 25600, 8, "column"), (ams.FP45, 16, 7168, 9728, 4, "slice"), (ams.FP433, 16, 7168, 13824, 4, "slice"),
        (ams.FP425, 8, 4096, 14336, 4, "slice"), (ams.FP533, 16, 5120, 25600, 4, "slice"),
    ],
)
def test_short_slices_of_a_split(fmt, M, N, K, slices, want):
    kind, p = plan(fmt, M, N, K, with_workspace=True)
    assert kind == want and int(p["k_slices"]) == slices, p


@pytest.mark.parametrize(
    "fmt,M,N,K,split",
    [
        (ams.FP533, 32, 5120, 6144, False), (ams.FP45, 16, 7168, 8192, False), (ams.FP533, 32, 5120, 9600, True),  # slices on column_kernel
        (ams.FP533, 7, 8714, 14560, False), (ams.FP533, 8, 8244, 13272, False), (ams.FP533, 12, 10612, 14552, False), (ams.FP425, 16, 9049, 16088, True),
        (ams.FP425, 12, 2187, 7848, True), (ams.FP45, 12, 2238, 7640, True), (ams.FP425, 12, 2187, 5000, False),  # on slice_kernel: K by the rows
        # up to 128 strips, where a plain call deals its rows: by the bytes a compute unit moves (1187 x 7848 split 6.4 us, whole 5.2)
        (ams.FP425, 12, 1187, 7848, False), (ams.FP45, 12, 1238, 7640, False), (ams.FP425, 12, 1187, 5000, False), (ams.FP425, 12, 1024, 14592, False), (ams.FP425, 12, 1024, 14600, True),
        (ams.FP425, 8, 2048, 13056, False), (ams.FP425, 8, 2048, 13064, True), (ams.FP533, 12, 2048, 10464, False), (ams.FP533, 12, 2048, 10472, True), (ams.FP425, 32, 1024, 12032, False), (ams.FP425, 32, 1024, 12040, True),
        (ams.FP533, 5, 1920, 9920, False), (ams.FP425, 5, 1920, 10960, False), (ams.FP425, 5, 1920, 16000, True), (ams.FP425, 16, 2560, 9208, False), (ams.FP425, 16, 2560, 9216, True),
        (ams.FP6, 9, 69, 7200, False), (ams.FP6, 9, 69, 7208, True), (ams.FP425, 12, 160, 10752, False), (ams.FP425, 12, 160, 10760, True),  # a few strips: less
        (ams.FP425, 32, 896, 2880, False), (ams.FP425, 32, 4096, 4096, False), (ams.FP533, 16, 1226, 5760, False),
    ],
)
def test_a_split_only_where_it_beats_the_plain_call(fmt, M, N, K, split):
    assert (plan(fmt, M, N, K, with_workspace=1)[1]["k_slices"] != "1") == split == (ams.ams_linear_workspace_bytes(fmt, M, N, K) > 0)
    if not split:
        assert plan(fmt, M, N, K, with_workspace=1) == plan(fmt, M, N, K)


def test_deep_and_two_strip_plans_stay_where_their_kernels_exist():
    # the kernels with three records ahead are built for M <= 16 (FP4.25: unaligned rows only), the ones with two strips
    # per wavefront for one row tile and formats without side groups
    rng = np.random.default_rng(20)
    deep = two = 0
    for _ in range(30000):
        fmt, M = int(rng.integers(7)), int(rng.integers(1, 33))
        N, K = 16 * int(rng.integers(1, 4500)), int(2 ** rng.uniform(3, 16))
        if rng.random() < 0.5:
            K = K // 8 * 8
        kind, p = plan(fmt, M, N, K, with_workspace=int(rng.integers(3)))
        if kind != "column":
            continue
        if p["strips_per_wave"] != "1":
            two += 1
            assert M <= 8 and fmt in (ams.FP533, ams.FP5, ams.FP4), (fmt, M, N, K, p)
        elif p["ahead"] != "2":
            deep += 1
            assert M <= 16 and (fmt in (ams.FP533, ams.FP5, ams.FP4) or (fmt == ams.FP425 and K % 8 and p["side_groups"] == "1")), (fmt, M, N, K, p)
    assert deep > 50 and two > 50


@pytest.mark.parametrize(
    "fmt,M,N,K,asks",
    [
        (ams.FP425, 1, 4096, 14336, dict(waves="16", ahead="1")),  # one strip: one record ahead
        (ams.FP425, 8, 4096, 14336, dict(waves="8", ahead="2", x_ahead="2")),
        (ams.FP425, 12, 4096, 4096, dict(waves="16", ahead="1", streams="12")),
        (ams.FP425, 1, 6144, 4096, dict(waves="16", ahead="2", streams="12")),  # two strips
        (ams.FP533, 1, 6144, 4096, dict(waves="16", ahead="2")),
        (ams.FP425, 8, 6144, 4096, dict(waves="8", ahead="2")),
        (ams.FP425, 1, 28672, 4096, dict(waves="8", ahead="3")),
        (ams.FP425, 3, 6144, 4099, dict(waves="16", ahead="2", streams="12", streamed_rows="3")),  # unaligned rows
        (ams.FP533, 5, 4096, 4099, dict(waves="16", ahead="1", streamed_rows="5")),
    ],
)
def test_a_slice_plan_says_what_its_kernel_asks_for(fmt, M, N, K, asks):
    kind, p = plan(fmt, M, N, K)
    assert kind == "slice" and {k: v for k, v in p.items() if k in ("waves", "ahead", "streams", "x_ahead", "streamed_rows")} == asks, p


@pytest.mark.parametrize(
    "fmt,M,strips,n_rec,deep",
    [
        (ams.FP533, 1, 160, 95, False), (ams.FP533, 1, 160, 96, True), (ams.FP533, 1, 223, 96, True), (ams.FP533, 1, 224, 96, False), (ams.FP533, 1, 1, 300, True),
        (ams.FP4, 2, 160, 159, False), (ams.FP4, 2, 160, 160, True), (ams.FP4, 3, 160, 300, False), (ams.FP5, 1, 160, 127, False), (ams.FP5, 1, 160, 128, True),
        (ams.FP5, 2, 160, 239, False), (ams.FP5, 2, 160, 240, True), (ams.FP425, 1, 160, 180, False), (ams.FP433, 1, 160, 180, False),
    ],
)
def test_one_strip_asks_for_two_records_ahead_where_that_is_faster(fmt, M, strips, n_rec, deep):
    K = n_rec * (96 if fmt in (ams.FP533, ams.FP433, ams.FP6) else 128)
    kind, p = plan(fmt, M, 16 * strips - 3, K - 8)
    assert kind == "slice" and (p["ahead"], p.get("x_ahead", "1")) == (("2", "2") if deep else ("1", "1")), p
    assert "x_ahead" not in plan(fmt, M, 16 * strips, K, with_workspace=2)[1]  # one scale per run


@pytest.mark.parametrize("M,N", [(9, 2300), (15, 4096), (20, 2000), (26, 2000)])  # 20 and 26 rows: two tiles
@pytest.mark.parametrize("fmt,last", [(ams.FP533, 28), (ams.FP433, 36), (ams.FP6, 28)])
def test_tiles_of_sixteen_rows_have_eight_wavefronts_where_twelve_leave_a_round_half_empty(fmt, last, M, N):
    for n_rec, deep in ((15, False), (16, True), (last, True), (last + 1, False)):
        kind, p = plan(fmt, M, N, 96 * n_rec - 8)
        assert kind == "slice" and p.get("row_tiles", "1") == ("2" if M > 16 else "1"), p
        want = ("8", "8", "2", "2") if deep else ("16", "12", "1", "1")
        assert (p["waves"], p.get("streams", p["waves"]), p["ahead"], p.get("x_ahead", "1")) == want, p
    assert plan(ams.FP425, M, N, 128 * 16)[1]["streams"] == "12"


@pytest.mark.parametrize("fmt", [ams.FP425, ams.FP45, ams.FP5, ams.FP4])
@pytest.mark.parametrize("entry", [0, GROUPED])
def test_eight_wavefronts_for_13_to_16_rows_of_128_weight_records(fmt, entry):
    for M, N, n_rec, deep in ((12, 3200, 18, False), (13, 3200, 17, False), (13, 3200, 18, True), (15, 3200, 18, True), (15, 3200, 200, True), (17, 3200, 18, False), (20, 2000, 18, False), (26, 2000, 18, True)):
        kind, p = plan(fmt, M, N, 128 * n_rec - 8, with_workspace=entry)
        assert kind == "slice" and ((p["strips_per_wg"], p["waves"], p.get("streams", ""), p.get("x_ahead", "")) == ("1", "8", "", "2")) == deep, p
