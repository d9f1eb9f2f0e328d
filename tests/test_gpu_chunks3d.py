"""One-step 3D launches where their blocks and chunks can go wrong: grids of
whole blocks and of one cell more, chunks of 4 and 8 planes with remainders,
blocks inside the grid beside ragged ones, receivers on every plane, more of
them on a plane than the workgroup has threads, some sharing a cell, and a
source on a chunk's first plane; against two steps per launch, bit for bit, and
the modelled data against the oracle."""
import numpy as np
import pytest
import torch

from oracle import core
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


# (nx, ny, nz, nb, shots): padded 128 x 32 x 32 (whole blocks and chunks),
# 129 x 33 x 33, a single ragged block, and a plan with 400 blocks of 8 planes
CASES = [(120, 24, 24, 4, 2), (121, 25, 25, 4, 2), (20, 11, 9, 5, 3), (57, 25, 17, 4, 60)]


@pytest.mark.parametrize("nx,ny,nz,nb,ns", CASES)
def test_one_step_chunks(esi, nx, ny, nz, nb, ns):
    rng = np.random.default_rng(51)
    nt = 9 if ns < 10 else 5
    vel = rng.uniform(1900.0, 2700.0, (nz, ny, nx)).astype(np.float32)
    spots = [(nx // 2, 4, ny // 2), (0, 0, 0), (nx - 1, nz - 1, ny - 1)]
    src = np.array([spots[s % 3] for s in range(ns)], dtype=np.int32)
    recs, ptr = [], [0]
    for s in range(ns):
        gy, gx = np.meshgrid(np.arange(ny), np.arange(nx), indexing="ij")
        r = [np.stack([gx.ravel(), np.full(gx.size, 2), gy.ravel()], 1)]          # a whole plane
        r += [np.stack([np.full(nz, nx // 3), np.arange(nz), np.full(nz, ny // 2)], 1)]   # every plane
        r += [np.array([[nx // 3, nz // 2, ny // 2]] * 2)]                         # and a shared cell
        if s == 1:
            r = [np.zeros((0, 3))]
        recs.append(np.concatenate(r).astype(np.int32))
        ptr.append(ptr[-1] + len(recs[-1]))
    plan = esi.Plan(ndim=3, nz=nz, ny=ny, nx=nx, nb=nb, nt=nt, dx=10.0, dt=1e-3, beta=1e-2, src=src,
                    rec_ptr=np.array(ptr), rec=np.concatenate(recs), vel=torch.from_numpy(vel).to(DEV))
    g = torch.Generator(device=DEV).manual_seed(6)
    w = torch.randn((ns, nt), generator=g, device=DEV)
    q = torch.randn(plan.vec_shape(ns), generator=g, device=DEV)
    d = torch.randn(plan.data_shape(), generator=g, device=DEV)

    def everything():
        gs = torch.zeros_like(w)
        return [plan.forward(w), plan.forward(q, esi.SRC_DENSE), plan.adjoint(d), plan.normal_apply(q)[0],
                plan.gradient(esi.GRAD_PENALTY, q),
                plan.gradient(esi.GRAD_SEED, w, d, kind=esi.SRC_POINT, grad_src=gs, ckpt_every=4), gs]

    one = everything()
    plan.set_time_block(2)
    two = everything()
    for k, (a, b) in enumerate(zip(one, two)):
        assert torch.equal(a, b), k
    grid = core.Grid(3, nz, nx, ny, nb=nb, nt=nt, dx=10.0, dt=1e-3)
    m = core.make_model(grid, vel)
    n0 = nt * len(recs[0])
    ref = core.forward(m, w[0].double().cpu().numpy(), recs[0], src_pos=src[0])
    got = one[0][:n0].cpu().numpy().reshape(nt, -1)
    # float32 fields over a few steps: rounding of 2^-24 a step and stencil arm
    assert np.linalg.norm(got - ref) < 1e-5 * np.linalg.norm(ref)
    plan.close()
