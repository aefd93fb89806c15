"""Products in 256x256 blocks at sizes that 256 and the 64-deep k-tiles do not
divide: the planner takes them for long reductions only, so each shape is large
enough for its product to be chosen (at these sizes: dW_ih and dW_hh over 6517
frames of a 224-cell layer, dz over 8001 classes, dW_s over 6013 frames).
bf16 tolerance of tests/test_gpu_parity.py."""

import pytest
import torch

from test_gpu_parity import BF16_TOL, run_step_and_compare

pytestmark = pytest.mark.gpu


def test_weight_gradients_ragged(gpu_lib):
    run_step_and_compare(dict(L=1, D=260, H=224, P=16, K=30, T=7, B=931), "bf16", BF16_TOL, dist="zipf", seed=31,
                         check_update=False)


@pytest.mark.parametrize("P,K,T,B", [(512, 8001, 3, 2871), (1024, 4001, 7, 859)])
def test_head_products_ragged(gpu_lib, P, K, T, B):
    """dz, dW_s and what follows from them against float64 on the GPU."""
    from paper_1907_05701_amd.step import LearnerStep

    H = 64
    print(f"[256x256] P={P} K={K} M={T * B}", flush=True)
    st = LearnerStep(L=1, D=8, H=H, P=P, K=K, T=T, B=B)
    g = torch.Generator(device="cuda").manual_seed(9)
    st.theta.copy_(torch.rand(st.theta.numel(), generator=g, device="cuda") * 0.2 - 0.1)
    st.pack()
    st.y_top.copy_(torch.rand(st.y_top.shape, generator=g, device="cuda") * 2 - 1)
    # skewed labels: the mean gradient is far from cancelling
    st.labels.copy_((K * torch.rand((T, B), generator=g, device="cuda") ** 4).to(torch.int32).clamp_(max=K - 1))
    st.grad.zero_()
    st.head()
    torch.cuda.synchronize()
    th = st.theta.double()
    n_head = P * 2 * H + P + K * P + K
    h = th[-n_head:]
    W_l, b_l = h[:P * 2 * H].view(P, 2 * H), h[P * 2 * H:P * 2 * H + P]
    W_s, b_s = h[P * 2 * H + P:-K].view(K, P), h[-K:]
    y = st.y_top.double().view(T * B, 2 * H)
    z = y @ W_l.t() + b_l
    s = z @ W_s.t() + b_s
    lab = st.labels.view(-1).long()
    ds = torch.softmax(s, 1)
    ds[torch.arange(T * B, device="cuda"), lab] -= 1.0
    ds /= T * B
    dz = ds @ W_s
    want = torch.cat([(dz.t() @ y).reshape(-1), dz.sum(0), (ds.t() @ z).reshape(-1), ds.sum(0)])
    got = st.grad[-n_head:].double()

    def rel(a, b):
        return float((a - b).norm() / b.norm())

    off = 0
    for name, size in (("W_l", P * 2 * H), ("b_l", P), ("W_s", K * P), ("b_s", K)):
        e = rel(got[off:off + size], want[off:off + size])
        print(f"[256x256] {name} {e:.2e}", flush=True)
        assert e <= BF16_TOL, name
        off += size
    assert rel(st.dy_top.double().view(T * B, 2 * H), dz @ W_l) <= BF16_TOL
    # row by row: a wrong row of an edge block scores about 1
    rows = (got[P * 2 * H + P:-K].view(K, P) - want[P * 2 * H + P:-K].view(K, P)).norm(dim=1)
    assert float((rows / want[P * 2 * H + P:-K].view(K, P).norm(dim=1)).max()) <= 0.2
    rows = (st.dy_top.double().view(T * B, 2 * H) - dz @ W_l).norm(dim=1)
    assert float((rows / (dz @ W_l).norm(dim=1)).max()) <= 0.2
