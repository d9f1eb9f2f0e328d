"""The WRI penalty gradient (point source and extended source together) on every
tile height of the two-step 2D launches against one-step launches, bit for bit."""
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


# the plan's own choice: 8-row tiles for 3 shots, 16-row tiles for 30, 24-row
# ones for 45; and the heights callers can set
@pytest.mark.parametrize("ns,shape", [(3, None), (30, None), (45, None), (3, 2), (3, 3), (3, 4)])
@pytest.mark.parametrize("nx,nz,nb", [(152, 88, 8), (153, 89, 8), (37, 70, 4)])
def test_penalty_gradient_bitwise(esi, nx, nz, nb, ns, shape):
    rng = np.random.default_rng(3)
    nt = 7
    src = np.stack([rng.integers(0, nx, ns), rng.integers(0, nz, ns)], 1).astype(np.int32)
    src[0] = (0, 0)
    src[1] = (nx - 1, nz - 1)
    rec = np.concatenate([np.stack([np.arange(nx), np.full(nx, 3)], 1)] * ns).astype(np.int32)
    vel = torch.from_numpy(rng.uniform(1900.0, 2700.0, (nz, nx)).astype(np.float32)).to(DEV)
    plan = esi.Plan(ndim=2, nz=nz, nx=nx, nb=nb, nt=nt, dx=10.0, dt=1e-3, beta=1e-2, src=src,
                    rec_ptr=np.arange(ns + 1) * nx, rec=rec, vel=vel)
    g = torch.Generator(device=DEV).manual_seed(5)
    w = torch.randn((ns, nt), generator=g, device=DEV)
    q = torch.randn(plan.vec_shape(ns), generator=g, device=DEV)
    plan.set_time_block(1)
    ref = plan.wri_gradient(esi.GRAD_PENALTY, w, q).clone()
    plan.set_time_block(2)
    if shape:
        plan.set_launch_shape(shape, shape)
    assert torch.equal(plan.wri_gradient(esi.GRAD_PENALTY, w, q), ref)
    plan.close()
