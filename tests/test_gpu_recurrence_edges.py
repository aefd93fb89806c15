"""The bf16 persistent recurrences against the float64 oracle where their plan
changes: a last member of 32 units (H no multiple of 64), 8, 16 and 32 rows per
workgroup with a partial last slice, groups padded to whole XCDs or not, two
launches per layer, and batches that 8 does not divide (the weight gradients
read da as it lies).  The tolerance is the bf16 path's (tests/test_gpu_parity.py)."""

import pytest

from test_gpu_parity import BF16_TOL, run_step_and_compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,T,B", [
    (32, 3, 1), (32, 5, 301),          # one member of 32 units; 16-row workgroups
    (96, 4, 9), (96, 3, 530),          # two members; two launches
    (160, 4, 203), (288, 3, 100),      # three and five members (five: groups not padded at this batch)
    (480, 3, 130), (480, 2, 517),      # eight members: 16-row workgroups, in one launch and in three
    (512, 3, 511), (512, 2, 61),       # 32-row workgroups with a partial quad, padded groups
    (192, 2, 1350),                    # 32-row workgroups in two launches
], ids=lambda v: str(v))
def test_recurrence_plan_edges(gpu_lib, H, T, B):
    run_step_and_compare(dict(L=2, D=20, H=H, P=16, K=30, T=T, B=B), "bf16", BF16_TOL, seed=23, check_update=False)


@pytest.mark.parametrize("rows", ["8", "16", "32"])
def test_fused_projection_with_a_partial_member(gpu_lib, monkeypatch, rows):
    """The forward computes the input projection itself (a choice made by the
    number of workgroups otherwise): same tolerance with a last member of 32
    units, at each number of rows per workgroup."""
    monkeypatch.setenv("ADPSGD_BLSTM_FUSE_GX", "1")
    monkeypatch.setenv("ADPSGD_BLSTM_ROWS_PER_WG", rows)
    run_step_and_compare(dict(L=2, D=20, H=160, P=16, K=30, T=13, B=50), "bf16", BF16_TOL, seed=29, check_update=False)
