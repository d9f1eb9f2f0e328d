"""One-step 3D launches on every chunk length the plan may choose (3 to 8
planes, with remainders): one step per launch against two, bit for bit."""
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


# on padded 64 x 16 x (nz + 8) grids the plan takes chunks of 3, 4, 5, 6, 7, 8 planes
@pytest.mark.parametrize("nz,ns", [(17, 20), (17, 29), (17, 37), (21, 86), (17, 57), (21, 103)])
def test_chunk_lengths(esi, nz, ns):
    nx, ny, nb, nt = 56, 8, 4, 4
    rng = np.random.default_rng(8)
    src = np.stack([rng.integers(0, nx, ns), rng.integers(0, nz, ns), rng.integers(0, ny, ns)], 1).astype(np.int32)
    gy, gx = np.meshgrid(np.arange(ny), np.arange(0, nx, 3), indexing="ij")
    one = np.concatenate([np.stack([gx.ravel(), np.full(gx.size, 2), gy.ravel()], 1),
                          np.stack([np.full(nz, 5), np.arange(nz), np.full(nz, 3)], 1)]).astype(np.int32)
    vel = torch.from_numpy(rng.uniform(1900.0, 2700.0, (nz, ny, nx)).astype(np.float32)).to(DEV)
    plan = esi.Plan(ndim=3, nz=nz, ny=ny, nx=nx, nb=nb, nt=nt, dx=10.0, dt=1e-3, beta=1e-2, src=src,
                    rec_ptr=np.arange(ns + 1) * len(one), rec=np.concatenate([one] * ns), vel=vel)
    g = torch.Generator(device=DEV).manual_seed(6)
    w = torch.randn((ns, nt), generator=g, device=DEV)
    d = torch.randn(plan.data_shape(), generator=g, device=DEV)

    def everything():
        return [plan.forward(w).clone(), plan.adjoint(d).clone(),
                plan.gradient(esi.GRAD_SEED, w, d, kind=esi.SRC_POINT, ckpt_every=2).clone()]

    first = everything()
    plan.set_time_block(2)
    for k, (a, b) in enumerate(zip(first, everything())):
        assert torch.equal(a, b), k
    plan.close()
