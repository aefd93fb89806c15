"""Workgroups of the persistent recurrences that wait for each other: groups
whose members do not all get to run are done by one workgroup, with the same
results bit for bit, so calls on several streams, graphs replayed side by side
and other work on the device never change or spoil a result."""

import threading

import pytest
import torch

pytestmark = pytest.mark.gpu


def _step(shape, precision, seed):
    from paper_1907_05701_amd.step import LearnerStep

    st = LearnerStep(**shape, precision=precision)
    g = torch.Generator(device="cuda").manual_seed(seed)
    st.grad.zero_()
    st.theta.copy_(torch.rand(st.theta.numel(), generator=g, device="cuda") * 0.2 - 0.1)
    st.pack()
    st.x.copy_(torch.randn(st.x.shape, generator=g, device="cuda"))
    dy = torch.randn((shape["T"], shape["B"], 2 * shape["H"]), generator=g, device="cuda") * 1e-3
    return st, dy


def _pass(st, dy):
    st.forward()
    st.backward(dy)


def _alone(st):
    """Whether a group ran on one workgroup since the last check_recurrence."""
    return bool(st.act_ws[-252:-248].view(torch.int32).item())


def _forced(st, dy, monkeypatch, **env):
    """Outputs of a pass as it is, and with members that never wait for their group."""
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    _pass(st, dy)
    st.check_recurrence()
    want = st.y_top.clone(), st.grad.clone()
    monkeypatch.setenv("ADPSGD_BLSTM_GROUP_WAIT_US", "0")
    st.y_top.zero_()
    st.grad.zero_()
    _pass(st, dy)
    torch.cuda.synchronize()
    alone = _alone(st)
    st.check_recurrence()
    monkeypatch.delenv("ADPSGD_BLSTM_GROUP_WAIT_US")
    assert torch.isfinite(want[0].float()).all() and torch.isfinite(want[1]).all()
    assert torch.equal(st.y_top, want[0]) and torch.equal(st.grad, want[1])
    return alone


@pytest.mark.parametrize("rows", ["8", "16", "32"])
@pytest.mark.parametrize("fuse", ["0", "1"])
@pytest.mark.parametrize("H,B", [(512, 61), (192, 77), (480, 37)])
def test_groups_on_one_workgroup_bf16(gpu_lib, monkeypatch, H, B, fuse, rows):
    """Every number of rows per workgroup, with the input projection inside the
    forward and dy as partial sums inside the backward, or not; whole and
    partial last members; partial slices."""
    print(f"[groups] bf16 H={H} B={B} fuse={fuse} rows={rows}", flush=True)
    st, dy = _step(dict(L=2, D=44, H=H, P=16, K=30, T=6, B=B), "bf16", 3)
    assert _forced(st, dy, monkeypatch, ADPSGD_BLSTM_ROWS_PER_WG=rows, ADPSGD_BLSTM_FUSE_GX=fuse,
                   ADPSGD_BLSTM_FUSE_DY=fuse)


@pytest.mark.parametrize("precision,H,B", [
    ("bf16", 288, 200), ("bf16", 448, 137), ("bf16", 96, 530),   # groups over several XCDs (twice), two launches a layer
    ("fp32", 144, 6), ("fp32", 256, 270), ("fp32", 432, 37), ("fp32", 512, 62), ("fp32", 512, 130),
], ids=lambda v: str(v))
def test_groups_on_one_workgroup_at_plan_edges(gpu_lib, monkeypatch, precision, H, B):
    print(f"[groups] {precision} H={H} B={B}", flush=True)
    st, dy = _step(dict(L=2, D=20, H=H, P=16, K=30, T=5, B=B), precision, 4)
    assert _forced(st, dy, monkeypatch)


@pytest.mark.parametrize("kinds", [("bf16", 512, "fp32", 512), ("bf16", 512, "bf16", 480), ("bf16", 512, "bf16", 512),
                                   ("fp32", 288, "bf16", 288)], ids=lambda k: "-".join(map(str, k)))
@pytest.mark.parametrize("graphs", [False, True], ids=["eager", "graphs"])
def test_two_streams_side_by_side(gpu_lib, kinds, graphs):
    """Two models on streams of their own, whose launches each want the whole
    chip: eagerly from two threads, and as graphs replayed on two streams."""
    print(f"[groups] two streams {kinds} graphs={graphs}", flush=True)
    steps, want, run = [], [], []
    streams = [torch.cuda.Stream() for _ in range(2)]
    for i in range(2):
        st, dy = _step(dict(L=2, D=40, H=kinds[2 * i + 1], P=16, K=30, T=9, B=128), kinds[2 * i], 41 + i)
        _pass(st, dy)
        steps.append((st, dy))
        want.append((st.y_top.clone(), st.grad.clone()))
        if graphs:
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                _pass(st, dy)
            run.append(graph.replay)
        else:
            run.append(lambda st=st, dy=dy: _pass(st, dy))
    torch.cuda.synchronize()
    for st, _ in steps:
        st.y_top.zero_()
        st.grad.zero_()
    torch.cuda.synchronize()

    def passes(i):
        with torch.cuda.stream(streams[i]):
            for _ in range(10):
                run[i]()

    threads = [threading.Thread(target=passes, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for (st, _), (y, grad) in zip(steps, want):
        st.check_recurrence()
        assert torch.equal(st.y_top, y) and torch.equal(st.grad, grad)
