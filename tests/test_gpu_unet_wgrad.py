"""Weight gradients of the network at the sizes where their tiles (64 pixels
wide, 2 to 8 rows, 16 or 32 channels) can go wrong: the smallest image, images
of whole tiles and of one pixel column of eight more at every level, and batches
whose tiles outnumber the chunks; against the oracle with bf16 rounding."""
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


@pytest.mark.parametrize("H,W,B,scale", [(8, 8, 1, 1.0), (64, 128, 1, 1.0), (72, 136, 3, 1.0), (16, 520, 2, 1e3)])
def test_weight_gradients(esi, H, W, B, scale):
    rng = np.random.default_rng(31)
    theta = inputs.he_init(ounet.fan_segments(), 31)
    theta[-17:] = rng.standard_normal(17).astype(np.float32) * 0.1
    x = rng.standard_normal((B, 3, H, W)).astype(np.float32)
    a = (scale * (rng.random((B, H, W)) + 0.05)).astype(np.float32)
    c = (scale * (rng.random((B, H, W)) * 0.5)).astype(np.float32)
    net = esi.Unet(H, W, B)
    net.set_params(torch.from_numpy(theta).to(DEV))
    t = [torch.from_numpy(v).to(DEV) for v in (x, a, c)]
    g, L = net.loss_grad(*t)
    g2, L2 = net.loss_grad(*t)
    assert torch.equal(g, g2) and L == L2            # sums in a fixed order
    o, cache = ounet.forward(theta.astype(np.float64), x.astype(np.float64), bf=True)
    L_ref, go = ounet.scaling_loss(o, a[:, None].astype(np.float64), c[:, None].astype(np.float64))
    g_ref = ounet.backward(theta.astype(np.float64), cache, go)
    g = g.cpu().numpy()
    assert abs(L - L_ref) < 5e-3 * abs(L_ref)
    # activations and their gradients are bf16 (half an ulp 2^-9): a layer's
    # float32 sums inherit the few per mille of those that round the other way
    off = 0
    for name, kind, ci, co in ounet.layers():
        n = int(np.prod(ounet._wshape(kind, ci, co))) + co
        assert np.linalg.norm(g[off:off + n] - g_ref[off:off + n]) < 2e-2 * np.linalg.norm(g_ref[off:off + n]), name
        off += n
    net.close()
