"""The float32 persistent recurrences against the float64 oracle, at the edges
of their plan: members of 128, 64 and 32 units (H up to 128, 256, 512) with a
partial last member, slices of 4, 8 and 16 rows with a partial last slice, more
than one launch per layer, one and two steps (both exchange slots).  The
tolerance is the float32 path's (tests/test_gpu_parity.py)."""

import pytest

from test_gpu_parity import FP32_TOL, run_step_and_compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,T,B", [
    (16, 3, 1), (32, 4, 300), (48, 2, 5), (64, 5, 700), (80, 3, 6), (128, 4, 9),   # one member, no exchange
    (128, 2, 1030),                                    # one member, 8-row slices, two launches
    (144, 3, 6), (240, 5, 130), (256, 3, 270),         # 64-unit members: partial last member, 4 and 8 rows, two launches
    (272, 1, 3), (272, 4, 33), (512, 3, 62), (512, 2, 130),   # 32-unit members: 4, 8 and 16 rows, two launches
    (288, 3, 52), (432, 3, 33),                        # nine members with 26 groups, fourteen with 18: the last two on several XCDs
], ids=lambda v: str(v))
def test_float32_recurrence_plan_edges(gpu_lib, H, T, B):
    run_step_and_compare(dict(L=2, D=24, H=H, P=16, K=30, T=T, B=B), "fp32", FP32_TOL, seed=17, check_update=False)


def test_float32_recurrence_many_steps(gpu_lib):
    run_step_and_compare(dict(L=1, D=8, H=288, P=8, K=10, T=70, B=7), "fp32", FP32_TOL, seed=18, check_update=False)


@pytest.mark.parametrize("shape", [
    dict(L=2, D=12, H=80, P=72, K=133, T=7, B=11),      # 77 frames, 133 classes (136 padded): partial blocks, k past whole chunks
    dict(L=2, D=36, H=144, P=40, K=260, T=33, B=2),     # 66 frames: a two-row block, k of two and a bit k-tiles
    dict(L=2, D=260, H=256, P=128, K=600, T=9, B=64),   # split dX and dz, whole blocks
], ids=lambda s: f"H{s['H']}_M{s['T'] * s['B']}")
def test_float32_products_at_block_edges(gpu_lib, shape):
    run_step_and_compare(shape, "fp32", FP32_TOL, seed=19)


@pytest.mark.parametrize("precision,H", [("fp32", 512), ("bf16", 480)])
def test_steps_on_two_streams(gpu_lib, precision, H):
    """Two models stepped by two threads on streams of their own: launches that
    need the whole chip take turns, no exchange wait gives up, and the outputs
    are those of the same passes alone, bit for bit."""
    import threading

    import torch

    from paper_1907_05701_amd.step import LearnerStep

    shape = dict(L=2, D=40, H=H, P=16, K=30, T=9, B=128)
    steps, streams = [], [torch.cuda.Stream() for _ in range(2)]
    for i in range(2):
        st = LearnerStep(**shape, precision=precision)
        g = torch.Generator(device="cuda").manual_seed(41 + i)
        st.grad.zero_()
        st.theta.copy_(torch.rand(st.theta.numel(), generator=g, device="cuda") * 0.2 - 0.1)
        st.pack()
        st.x.copy_(torch.randn(st.x.shape, generator=g, device="cuda"))
        dy = torch.randn((shape["T"], shape["B"], 2 * H), generator=g, device="cuda") * 1e-3
        steps.append((st, dy))
    want = []
    for st, dy in steps:
        st.forward()
        st.backward(dy)
        want.append((st.y_top.clone(), st.grad.clone()))
    torch.cuda.synchronize()

    def passes(i):
        st, dy = steps[i]
        with torch.cuda.stream(streams[i]):
            for _ in range(10):
                st.forward()
                st.backward(dy)

    threads = [threading.Thread(target=passes, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for (st, _), (y, grad) in zip(steps, want):
        st.check_recurrence()
        assert torch.equal(st.y_top, y) and torch.equal(st.grad, grad)
