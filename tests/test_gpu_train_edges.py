"""GPU tests of the training step's two kernels at the edges of their tiles,
32-row slices and splits."""
import numpy as np
import pytest
import torch

from gpu_helpers import DEV

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pn():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from paper_1802_00147_amd import pn as P
    P.lib()
    return P


def inputs(pn, seed, rows=9000):
    from paper_1802_00147_amd import workloads as W
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    feat = torch.randn(rows, 8, generator=g, device=DEV)
    feat[:, 7] = 0.0
    lab = (torch.rand(rows, generator=g, device=DEV) < 0.3).float()
    tgt = torch.randn(rows, generator=g, device=DEV)
    idx = torch.randperm(rows, generator=g, device=DEV).to(torch.int32)
    params = W.mlp_init_weights(50)
    return pn.Network([w for w, _ in params], [b + 0.05 for _, b in params], DEV), feat, lab, tgt, idx


def bf(t):
    return t.view(torch.bfloat16).double()


# Tiles of 16 rows, slices of 32, splits from 512 rows, more than 16 splits of
# the outer layers from 2,176.
@pytest.mark.parametrize("B", [15, 16, 31, 32, 33, 48, 511, 513, 1000, 2177, 8200])
def test_gradients_from_a_used_workspace(pn, B):
    """The first step's moments against FP64 products of the step's own
    tensors, in a workspace full of NaN patterns (the padding rows of the last
    slice must be written): FP32 sums of exact bfloat16 products, 1e-5 of
    sum |g a|."""
    net, feat, lab, tgt, idx = inputs(pn, 61)
    ws = torch.full((int(pn.lib().pn_mlp_train_workspace_size(B)),), 0xFF, dtype=torch.uint8, device=DEV)
    loss = torch.zeros(1, device=DEV)
    pn.mlp_train_step(net, feat, lab, tgt, idx[:B].contiguous(), 1e-3, loss, ws)
    T = pn.mlp_train_step_tensors(ws, B)
    a = [bf(T["X"])[:, :7], bf(T["h1"]), bf(T["h2"]), bf(T["h3"])]
    g = [bf(T[k]) for k in ("g1", "g2", "g3", "g4")]
    assert np.isfinite(loss.item())
    for l in range(4):
        assert torch.all((net.mw[l].double() / 0.1 - g[l].T @ a[l]).abs() <= 1.1e-5 * (g[l].abs().T @ a[l].abs()) + 1e-30), l
        assert torch.all((net.mb[l].double() / 0.1 - g[l].sum(0)).abs() <= 1.1e-5 * g[l].abs().sum(0) + 1e-30), l


@pytest.mark.parametrize("B", [17, 700])
def test_weight_copies_follow_the_updates(pn, B):
    """Five steps of one call (the weights' other layouts kept by the updates)
    and five calls (formed anew from the bfloat16 weights): the same bits, with
    the bfloat16 weights the rounded FP32 ones."""
    one, feat, lab, tgt, idx = inputs(pn, 62)
    many = inputs(pn, 62)[0]
    loss = torch.zeros(1, device=DEV)
    pn.mlp_train(one, feat, lab, tgt, idx[:5 * B].contiguous(), B, 1e-3, loss)
    for b in range(5):
        pn.mlp_train_step(many, feat, lab, tgt, idx[b * B:(b + 1) * B].contiguous(), 1e-3, loss)
    for l in range(4):
        for x, y in ((one.w, many.w), (one.b, many.b), (one.vw, many.vw), (one.mb, many.mb)):
            assert torch.equal(x[l].view(torch.int32), y[l].view(torch.int32)), l
        assert torch.equal(one.wb[l].view(torch.bfloat16), one.w[l].to(torch.bfloat16)), l


@pytest.mark.parametrize("B", [33, 2048, 3600])
def test_last_step_leaves_its_tensors(pn, B):
    """Three steps of one call leave the third step's tensors in the workspace,
    as a single step from the same weights does: the same bits."""
    one, feat, lab, tgt, idx = inputs(pn, 63, rows=12000)
    many = inputs(pn, 63, rows=12000)[0]
    loss = torch.zeros(1, device=DEV)
    ws = pn.mlp_train(one, feat, lab, tgt, idx[:3 * B].contiguous(), B, 1e-3, loss)
    for b in range(3):
        ws1 = pn.mlp_train_step(many, feat, lab, tgt, idx[b * B:(b + 1) * B].contiguous(), 1e-3, loss)
    a, c = pn.mlp_train_step_tensors(ws, B), pn.mlp_train_step_tensors(ws1, B)
    for k in a:
        assert torch.equal(a[k].view(torch.int32 if k == "out" else torch.int16), c[k].view(torch.int32 if k == "out" else torch.int16)), k
