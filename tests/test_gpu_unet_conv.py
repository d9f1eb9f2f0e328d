"""The network's convolutions with fused first, pooling and last layers: images
smaller than a tile, of whole tiles, with a remainder of one group of pixels at
every level, and batches whose tiles outnumber the resident workgroups, so that
one walks several."""
import numpy as np
import pytest
import torch

from oracle import unet as ounet
from paper_2211_06300_amd import inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def esi():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2211_06300_amd import esi as e
    e.load_library()
    return e


def _net(esi, H, W, B):
    theta = inputs.he_init(ounet.fan_segments(), 37)
    theta[-17:] = np.random.default_rng(37).standard_normal(17).astype(np.float32) * 0.1
    net = esi.Unet(H, W, B)
    net.set_params(torch.from_numpy(theta).to(DEV))
    return net, theta


@pytest.mark.parametrize("H,W,B", [(8, 8, 1), (64, 128, 1), (72, 136, 3), (16, 520, 2)])
def test_forward_against_oracle(esi, H, W, B):
    net, theta = _net(esi, H, W, B)
    x = np.random.default_rng(5).standard_normal((B, 3, H, W)).astype(np.float32)
    o = net.forward(torch.from_numpy(x).to(DEV)).cpu().numpy()
    ref, _ = ounet.forward(theta.astype(np.float64), x.astype(np.float64), bf=True)
    # activations are bf16 (half an ulp 2^-9): float32 sums round a few per mille
    # of them the other way than float64 ones
    assert np.linalg.norm(o.ravel() - ref.ravel()) < 2e-2 * np.linalg.norm(ref)
    net.close()


@pytest.mark.parametrize("H,W,B", [(408, 808, 8), (200, 264, 24)])
def test_forward_of_many_tiles(esi, H, W, B):
    # an image's result does not depend on its batch: the same sums in the same order
    net, _ = _net(esi, H, W, B)
    x = torch.randn(B, 3, H, W, device=DEV, generator=torch.Generator(device=DEV).manual_seed(6))
    o = net.forward(x).clone()
    for _ in range(3):
        assert torch.equal(net.forward(x), o)
    for b in (0, B // 2, B - 1):
        assert torch.equal(net.forward(x[b:b + 1].contiguous()).reshape(-1), o[b].reshape(-1))
    net.close()


def test_training_forward_is_the_same(esi):
    # the training pass keeps every activation, the other forms neither the padded
    # input nor the last activation: the loss is that of the same output
    H, W, B = 72, 136, 3
    net, _ = _net(esi, H, W, B)
    rng = np.random.default_rng(7)
    x = torch.from_numpy(rng.standard_normal((B, 3, H, W)).astype(np.float32)).to(DEV)
    a = (rng.random((B, H, W)) + 0.05).astype(np.float32)
    c = (rng.random((B, H, W)) * 0.5).astype(np.float32)
    _, L = net.loss_grad(x, torch.from_numpy(a).to(DEV), torch.from_numpy(c).to(DEV))
    o = net.forward(x).cpu().numpy().reshape(B, 1, H, W).astype(np.float64)
    L_ref, _ = ounet.scaling_loss(o, a[:, None].astype(np.float64), c[:, None].astype(np.float64))
    # terms of the loss are float32 (2^-24 each), summed in float64
    assert abs(L - L_ref) < 1e-5 * abs(L_ref)
    net.close()
