"""FWI gradients whose segment store outgrows the last-level cache (two-step 2D
launches write and read it past the caches) against one-step launches, bit for
bit, on tiles of every height that large launches take."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def esi():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2211_06300_amd import esi as e
    e.load_library()
    return e


# 20 shots x 12 slots of 601 x 481 cells: 278 MB; of 601 x 321: 185 MB (kept)
@pytest.mark.parametrize("nz,shape", [(481, None), (481, 3), (481, 4), (321, None)])
def test_streamed_store(esi, nz, shape):
    nx, ns, nt, nb = 601, 20, 13, 8
    rng = np.random.default_rng(3)
    src = np.stack([rng.integers(0, nx, ns), rng.integers(0, nz, ns)], 1).astype(np.int32)
    rec = np.concatenate([np.stack([np.arange(0, nx, 2), np.full(301, 3)], 1)] * ns).astype(np.int32)
    vel = torch.from_numpy(rng.uniform(1900.0, 2700.0, (nz, nx)).astype(np.float32)).to(DEV)
    plan = esi.Plan(ndim=2, nz=nz, nx=nx, nb=nb, nt=nt, dx=10.0, dt=1e-3, beta=1e-2, src=src,
                    rec_ptr=np.arange(ns + 1) * 301, rec=rec, vel=vel)
    g = torch.Generator(device=DEV).manual_seed(5)
    w = torch.randn((ns, nt), generator=g, device=DEV)
    d = torch.randn(plan.data_shape(), generator=g, device=DEV)

    def gradient():
        return plan.gradient(esi.GRAD_SEED, w, d, kind=esi.SRC_POINT, ckpt_every=12).clone()

    plan.set_time_block(1)
    ref = gradient()
    plan.set_time_block(2)
    if shape:
        plan.set_launch_shape(shape, shape)
    assert torch.equal(gradient(), ref)
    plan.close()
