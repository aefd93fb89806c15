"""Dims whose head workspace lies just below the static entry point's 64 MiB:
split-K partials are part of that workspace, so a plan that splits further
would turn calls away that are accepted today."""

import pytest


@pytest.mark.parametrize("precision,H,P,K,T,B", [
    ("fp32", 416, 192, 8015, 95, 15), ("fp32", 544, 512, 3114, 3, 965), ("fp32", 320, 120, 10003, 1, 1156),
    ("fp32", 448, 144, 6473, 55, 35), ("bf16", 512, 256, 32000, 21, 30), ("bf16", 512, 256, 192, 300, 49),
    ("bf16", 64, 512, 1000, 40, 132), ("bf16", 96, 8, 9000, 60, 50)])
def test_dims_below_the_limit_stay_below_it(precision, H, P, K, T, B):
    from paper_1907_05701_amd import binding as bd
    dims = bd.make_dims(1, 8, H, P, K, T, B, precision)
    assert bd.blstm_workspace_bytes(dims)["head_ws"] <= bd.HEAD_STATIC_SCRATCH_BYTES
