"""Which kernel a Linear gets where the choice was measured to matter: shapes on which slice_kernel was the slower one
stay on column_kernel, and slice_kernel's workgroups keep the sizes that its rules assume.  Host only."""

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
