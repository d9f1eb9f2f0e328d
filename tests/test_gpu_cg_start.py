"""Start of a CG solve (direction, zero solution and squared norm of the right-hand
side in one pass) for vectors whose length is no multiple of four, for one shot
and several, and into buffers that hold other values: the first iterate is the
steepest-descent step."""
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


@pytest.mark.parametrize("nx,nz,nt,ns", [(37, 29, 11, 3), (36, 28, 12, 3), (21, 11, 5, 1)])
def test_first_iterate(esi, nx, nz, nt, ns):
    src = np.array([[nx // 2, 1 + s] for s in range(ns)], dtype=np.int32)
    rec = np.concatenate([np.stack([np.arange(nx), np.full(nx, 2)], 1)] * ns).astype(np.int32)
    vel = torch.full((nz, nx), 2200.0, device=DEV)
    plan = esi.Plan(ndim=2, nz=nz, nx=nx, nb=5, nt=nt, dx=10.0, dt=1e-3, beta=1e-2, src=src,
                    rec_ptr=np.arange(ns + 1) * nx, rec=rec, vel=vel)
    g = torch.Generator(device=DEV).manual_seed(2)
    d = torch.randn(plan.data_shape(), generator=g, device=DEV)
    x = torch.full(plan.vec_shape(ns), 7.0, device=DEV)
    work = torch.full((3, *plan.vec_shape(ns)), 5.0, device=DEV)
    b = plan.adjoint(d).double()
    x1, _ = plan.cg_solve(d, 1, x=x, work=work)
    Nb = plan.normal_apply(b.float())[0].double()
    for s in range(ns):   # x_1 = alpha b with alpha = b.b / b.N b
        al = float((b[s] * b[s]).sum() / (b[s] * Nb[s]).sum())
        # alpha from float32 fields over nt steps; one rounding of the update
        assert torch.linalg.norm(x1[s].double() - al * b[s]) < 1e-4 * torch.linalg.norm(al * b[s])
    plan.close()
