"""The bf16 persistent recurrences against the float64 oracle where their plan
changes: a last member of 32 units (H no multiple of 64), 8, 16 and 32 rows per
workgroup with a partial last slice, groups padded to whole XCDs or not, several
launches per layer whose last has rows per workgroup of its own, and batches
that 8 does not divide (the weight gradients read da as it lies).  The tolerance
is the bf16 path's (tests/test_gpu_parity.py)."""

import pytest

from test_gpu_parity import BF16_TOL, run_step_and_compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,T,B", [
    (32, 3, 1), (32, 5, 301),          # one member of 32 units
    (96, 4, 9), (96, 3, 530),          # two members; 16-row workgroups
    (160, 4, 203), (288, 3, 100),      # three and five members (groups padded to 32)
    (288, 3, 200), (448, 3, 137),      # five members with 50 groups, seven with 36: the last two and four on several XCDs
    (320, 3, 850),                     # the same with 32-row workgroups, in two launches (50 groups, then 4)
    (480, 3, 130), (480, 2, 517),      # eight members: 16-row workgroups, in one launch and in two and one of 8-row ones
    (480, 6, 400),                     # 16-row workgroups in both launches (fewer steps run one launch each)
    (512, 3, 511), (512, 2, 61),       # 32-row workgroups with a partial quad, padded groups
    (512, 3, 524), (512, 3, 700),      # launches of 32-row workgroups, then of 8-row and of 16-row ones
    (192, 2, 1350), (64, 3, 300),      # 32-row workgroups, then 8-row ones; 38 slices of one member
], ids=lambda v: str(v))
def test_recurrence_plan_edges(gpu_lib, H, T, B):
    run_step_and_compare(dict(L=2, D=20, H=H, P=16, K=30, T=T, B=B), "bf16", BF16_TOL, seed=23, check_update=False)


@pytest.mark.parametrize("rows,H", [("8", 160), ("16", 160), ("32", 192)])
def test_fused_projection_with_a_partial_member(gpu_lib, monkeypatch, rows, H):
    """The forward computes the input projection itself (a choice made by the
    number of workgroups and steps otherwise): same tolerance with a last member
    of 32 units, at each number of rows per workgroup that such widths take, and
    with whole members at 32 rows."""
    monkeypatch.setenv("ADPSGD_BLSTM_FUSE_GX", "1")
    monkeypatch.setenv("ADPSGD_BLSTM_ROWS_PER_WG", rows)
    run_step_and_compare(dict(L=2, D=20, H=H, P=16, K=30, T=13, B=50), "bf16", BF16_TOL, seed=29, check_update=False)


def test_layer_input_past_the_range_of_a_buffer_resource(gpu_lib, monkeypatch):
    """131072 frames of 8200 features: 2.15 GB in bf16, past the 2^31 bytes that
    one buffer resource reaches. The forward, which at this many workgroups
    computes the projection itself where it can, gives what the separate product
    gives, bit for bit (its resources are based on each block)."""
    import torch

    from paper_1907_05701_amd.step import LearnerStep

    st = LearnerStep(L=1, D=8200, H=192, P=8, K=10, T=2, B=65536)
    g = torch.Generator(device="cuda").manual_seed(7)
    st.theta.copy_(torch.rand(st.theta.numel(), generator=g, device="cuda") * 0.02 - 0.01)
    st.pack()
    st.x.normal_(generator=g)
    st.forward()
    got = st.y_top.clone()
    monkeypatch.setenv("ADPSGD_BLSTM_FUSE_GX", "0")
    st.y_top.zero_()
    st.forward()
    st.check_recurrence()
    assert torch.equal(got, st.y_top)
    assert got[-1, -64:].float().abs().mean() > 0.05   # (near zero with an input that reads as zeros)


@pytest.mark.parametrize("precision,H", [("bf16", 32), ("bf16", 96), ("bf16", 480), ("fp32", 64), ("fp32", 144)])
def test_a_nan_reaches_every_unit_one_step_later(gpu_lib, precision, H):
    """One unit's NaN (its forward-direction input bias) spreads through W_hh: at
    the first step that unit alone, from the second on every unit of that
    direction, whichever workgroup owns it; the other direction stays finite."""
    import torch

    from paper_1907_05701_amd.step import LearnerStep

    D, T, B = 8, 4, 9
    st = LearnerStep(L=1, D=D, H=H, P=8, K=10, T=T, B=B, precision=precision)
    g = torch.Generator(device="cuda").manual_seed(5)
    st.theta.copy_(torch.rand(st.theta.numel(), generator=g, device="cuda") * 0.2 - 0.1)
    unit = H - 3
    st.theta[4 * H * D + 4 * H * H + unit] = float("nan")   # b_ih of gate i
    st.pack()
    st.x.normal_(generator=g)
    st.forward()
    st.check_recurrence()
    bad = torch.isnan(st.y_top.float())
    want = torch.zeros_like(bad)
    want[0, :, unit] = True
    want[1:, :, :H] = True
    assert torch.equal(bad, want)
