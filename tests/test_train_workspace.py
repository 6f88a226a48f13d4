"""The training workspace: its size, and steps whose row-block tensors take the
places of the reported ones (more than 5,504 rows)."""
import numpy as np
import pytest

ROOM = 17576960        # bytes behind the reported tensors, whatever the batch


@pytest.fixture(scope="module")
def pn():
    from paper_1802_00147_amd import pn as P
    P.lib()
    return P


def al(x):
    return (x + 255) // 256 * 256


@pytest.mark.parametrize("batch", [1, 33, 2048, 4096, 5504, 5505, 5536, 8192, 65536, 1 << 20, (1 << 31) - 1])
def test_room_behind_the_tensors_does_not_grow(pn, batch):
    """A workspace of the size that the reported tensors and the fixed room
    take is enough for every batch; the assisted scan's grows by no more."""
    size = int(pn.lib().pn_mlp_train_workspace_size(batch))
    assert size == pn.mlp_train_workspace_layout(batch)[8] + al(batch * 512) + ROOM
    scan = [int(pn.lib().pn_surrogate_scan_workspace_size(1000, b)) for b in (batch, 1)]
    assert scan[0] - scan[1] == size - int(pn.lib().pn_mlp_train_workspace_size(1))


def inputs(pn, rows):
    import torch
    from gpu_helpers import DEV
    from paper_1802_00147_amd import workloads as W
    g = torch.Generator(device=DEV)
    g.manual_seed(71)
    feat = torch.randn(rows, 8, generator=g, device=DEV)
    feat[:, 7] = 0.0
    lab = (torch.rand(rows, generator=g, device=DEV) < 0.3).float()
    tgt = torch.randn(rows, generator=g, device=DEV)
    idx = torch.randperm(rows, generator=g, device=DEV).to(torch.int32)

    def net():
        params = W.mlp_init_weights(50)
        return pn.Network([w for w, _ in params], [b + 0.05 for _, b in params], DEV)
    return net, feat, lab, tgt, idx, torch.zeros(1, device=DEV)


def bits(t):
    import torch
    return t.view(torch.int32 if t.dtype == torch.float32 else torch.int16)


# The last batch with its own room, the first without (one row in the last
# slice), whole slices only, 8-row blocks cut at 7 and 1 rows, one tile past a slice.
@pytest.mark.gpu
@pytest.mark.parametrize("B", [5504, 5505, 5536, 5551, 8200, 8209])
def test_step_in_a_workspace_of_the_stated_size(pn, B):
    """Tensors, gradients and the workspace's end after a step in a workspace
    full of NaN patterns: the forward tensors are those of its halves bit for
    bit, g3, g2, g1 the masked products of the step's own tensors (FP32 sums of
    exact products rounded to bfloat16: 2^-8 of the value and 1e-5 of sum |g w|),
    the first moments 0.1 times the FP64 products (1e-5 of sum |g a|, and the
    rounding of the moment), and no byte behind the workspace changes."""
    import torch
    from gpu_helpers import DEV
    net, feat, lab, tgt, idx, loss = inputs(pn, 9000)
    need = int(pn.lib().pn_mlp_train_workspace_size(B))
    buf = torch.full((need + 65536,), 0xFF, dtype=torch.uint8, device=DEV)
    n = net()
    W = [w.view(torch.bfloat16).double().reshape(o, i) for w, o, i in zip([w.clone() for w in n.wb], (256, 256, 256, 2), (7, 256, 256, 256))]
    pn.mlp_train_step(n, feat, lab, tgt, idx[:B].contiguous(), 1e-3, loss, buf[:need])
    assert torch.all(buf[need:] == 0xFF)
    T = pn.mlp_train_step_tensors(buf, B)
    half = B // 2
    for lo, hi in ((0, half), (half, B)):
        ws = pn.mlp_train_step(net(), feat, lab, tgt, idx[lo:hi].contiguous(), 1e-3, loss)
        P = pn.mlp_train_step_tensors(ws, hi - lo)
        for k in ("X", "h1", "h2", "h3", "out"):
            assert torch.equal(bits(T[k][lo:hi]), bits(P[k])), (k, lo)
    D = {k: T[k].view(torch.bfloat16).double() for k in T if k != "out"}
    x, i = T["out"].double(), idx[:B].long()
    g4 = torch.stack([torch.sigmoid(x[:, 0]) - lab[i].double(), (x[:, 1] - tgt[i].double()).clamp(-1, 1)], 1) / B
    assert torch.all((D["g4"] - g4).abs() <= 2.0 ** -8 * g4.abs() + 1e-6 / B)
    for l, (g, up, h) in enumerate((("g1", "g2", "h1"), ("g2", "g3", "h2"), ("g3", "g4", "h3"))):
        keep = (D[h] > 0).double()
        ref, scale = (D[up] @ W[l + 1]) * keep, (D[up].abs() @ W[l + 1].abs()) * keep
        assert torch.all((D[g] - ref).abs() <= 2.0 ** -8 * ref.abs() + 1.1e-5 * scale), g
    a = [D["X"][:, :7], D["h1"], D["h2"], D["h3"]]
    for l in range(4):
        g = D["g%d" % (l + 1)]
        assert torch.all((n.mw[l].double() / 0.1 - g.T @ a[l]).abs() <= 1.1e-5 * (g.abs().T @ a[l].abs()) + 1e-30), l
        assert torch.all((n.mb[l].double() / 0.1 - g.sum(0)).abs() <= 1.1e-5 * g.abs().sum(0) + 1e-30), l
    assert np.isfinite(loss.item())


@pytest.mark.gpu
@pytest.mark.parametrize("B", [5504, 5505, 8200])
def test_steps_of_one_call_leave_the_last_ones_tensors(pn, B):
    """Three steps of one call and three calls: the same bits in the weights,
    the moments and the tensors left behind."""
    import torch
    net, feat, lab, tgt, idx, loss = inputs(pn, 3 * 8200)
    one, many = net(), net()
    ws = pn.mlp_train(one, feat, lab, tgt, idx[:3 * B].contiguous(), B, 1e-3, loss)
    for b in range(3):
        ws1 = pn.mlp_train_step(many, feat, lab, tgt, idx[b * B:(b + 1) * B].contiguous(), 1e-3, loss)
    p, q = pn.mlp_train_step_tensors(ws, B), pn.mlp_train_step_tensors(ws1, B)
    for k in p:
        assert torch.equal(bits(p[k]), bits(q[k])), k
    for x, y in ((one.w, many.w), (one.b, many.b), (one.mw, many.mw), (one.vb, many.vb)):
        for l in range(4):
            assert torch.equal(x[l].view(torch.int32), y[l].view(torch.int32)), l
