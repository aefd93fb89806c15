"""Upper bounds on act_ws: da is kept for every layer (the weight gradients of
all layers run in one launch at the end), but the top layer's takes the place of
the forward's input projection, so a model of one layer needs none for it."""

import pytest


@pytest.mark.parametrize("L,D,H,P,K,T,B,precision,mb", [
    (6, 260, 512, 256, 32000, 21, 128, "fp32", 785), (6, 260, 512, 256, 32000, 21, 128, "bf16", 472),
    (6, 260, 512, 256, 32000, 21, 100, "bf16", 377), (1, 260, 480, 24, 133, 21, 513, "bf16", 410),
    (1, 260, 480, 24, 133, 21, 128, "fp32", 190)])
def test_act_ws_below(L, D, H, P, K, T, B, precision, mb):
    from paper_1907_05701_amd import binding as bd
    got = bd.blstm_workspace_bytes(bd.make_dims(L, D, H, P, K, T, B, precision))["act_ws"] / 1e6
    print(f"{got:.1f} MB")
    assert got <= mb
