"""GPU test of the fused inference at each length of a workgroup's run of tiles:
its hidden activations rotate through three buffers."""
import pytest
import torch

from gpu_helpers import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles,more,short", [(2, 0, 0), (3, 0, 1), (4, 0, 1), (5, 3, 7), (7, 0, 31), (3, 1, 0)])
def test_runs_of_tiles_per_workgroup(tiles, more, short):
    """`tiles` 32-row tiles in every workgroup, one more in the first `more`,
    the last one short: the drain meets each of the three buffers (the last
    tile's index modulo 3 is 0, 1 and 2), and the outputs are the layer-wise
    path's bits."""
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from paper_1802_00147_amd import pn, workloads as W
    n = 32 * (tiles * torch.cuda.get_device_properties(0).multi_processor_count + more) - short
    g = torch.Generator(device=DEV)
    g.manual_seed(90 + n)
    feat = torch.randn(n, 8, generator=g, device=DEV)
    feat[:, 7] = 0.0
    params = W.mlp_init_weights(50)
    net = pn.Network([w for w, _ in params], [b + 0.05 for _, b in params], DEV)
    a, b = pn.mlp_infer(net, feat, chunk=1 << 14), pn.mlp_infer_fused(net, feat)
    assert torch.equal(a.view(torch.int32), b.view(torch.int32))
