"""Two-step 2D launches on every tile height against one-step launches, bit
for bit, at the sizes where their tiles can go wrong: grids of whole tiles and
one cell more, tiles wholly inside the grid beside ragged ones, sources and
receivers on tile borders, more receivers in a tile than the workgroup has
threads, and receivers sharing a cell.  (The one-step kernel is checked
against the oracle in test_gpu_parity.py.)"""
import numpy as np
import pytest
import torch

from paper_2211_06300_amd import inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (nx, nz, nb): padded widths of 3 and 3 1/56 tiles, heights of 13 and 13 1/8
# eight-row tiles (6.5 of 16, 4.3 of 24, 3.25 of 32, 2.6 of 40), and a grid of
# one ragged tile column
GRIDS = [(152, 88, 8), (153, 89, 8), (37, 70, 4)]
# shapes callers can set, and the plan's own choice: 8-row tiles for few
# shots, 16-row tiles for 60
SHAPES = [("set", 2), ("set", 3), ("set", 4), ("few", 2), ("many", 2)]


@pytest.fixture(scope="module")
def esi():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2211_06300_amd import esi as e
    e.load_library()
    return e


def _plan(esi, nx, nz, nb, ns, nt, seed):
    rng = np.random.default_rng(seed)
    # sources in the physical corners, on tile borders and inside
    spots = [(0, 0), (nx - 1, nz - 1), (min(56, nx - 1), min(32, nz - 1)), (min(55 - nb, nx - 1), 24 - nb),
             (nx // 2, nz // 2)]
    src = np.array([spots[s % len(spots)] for s in range(ns)], dtype=np.int32)
    ptr, recs = [0], []
    for s in range(ns):
        r = [np.stack([np.arange(nx), np.full(nx, 3)], 1)]           # a row across every tile column
        if s == 0:                                                   # a block of 400 cells, some of them twice
            gx, gz = np.meshgrid(np.arange(8, 28), np.arange(30, 50))
            r += [np.stack([gx.ravel(), gz.ravel()], 1), np.array([[9, 31], [9, 31], [27, 49]])]
        if s == 2:
            r = [np.zeros((0, 2))]                                   # a shot without receivers
        recs.append(np.concatenate(r).astype(np.int32))
        ptr.append(ptr[-1] + len(recs[-1]))
    vel = torch.from_numpy(rng.uniform(1900.0, 2700.0, (nz, nx)).astype(np.float32)).to(DEV)
    return esi.Plan(ndim=2, nz=nz, nx=nx, nb=nb, nt=nt, dx=10.0, dt=1e-3, beta=1e-2, src=src,
                    rec_ptr=np.array(ptr), rec=np.concatenate(recs), vel=vel)


def _everything(esi, plan, nt, ns):
    g = torch.Generator(device=DEV).manual_seed(5)
    w = torch.randn((ns, nt), generator=g, device=DEV)
    q = torch.randn(plan.vec_shape(ns), generator=g, device=DEV)
    d = torch.randn(plan.data_shape(), generator=g, device=DEV)
    gsrc = torch.zeros_like(w)
    out = [plan.forward(w), plan.forward(q, esi.SRC_DENSE), plan.adjoint(d), plan.normal_apply(q)[0],
           plan.gradient(esi.GRAD_PENALTY, q),
           plan.gradient(esi.GRAD_SEED, w, d, kind=esi.SRC_POINT, grad_src=gsrc, ckpt_every=5), gsrc]
    x, _ = plan.cg_solve(d, 3)
    return out, x


@pytest.mark.parametrize("how,shape", SHAPES)
@pytest.mark.parametrize("nx,nz,nb", GRIDS)
def test_two_step_tiles_bitwise(esi, nx, nz, nb, how, shape):
    ns, nt = (60, 7) if how == "many" else (3, 13)
    plan = _plan(esi, nx, nz, nb, ns, nt, 40)
    plan.set_time_block(1)
    ref, xref = _everything(esi, plan, nt, ns)
    plan.set_time_block(2)
    if how == "set":
        plan.set_launch_shape(shape, shape)
    got, x = _everything(esi, plan, nt, ns)
    for k, (a, b) in enumerate(zip(ref, got)):
        assert torch.equal(a, b), k
    # the dot products sum float64 partials over other tiles: alpha and beta
    # may differ in their last float64 bits, by one float32 bit once rounded
    # for the updates, and three updates of x and r follow
    assert float(torch.linalg.norm(x - xref)) <= 3 * 2 ** -23 * 4 * float(torch.linalg.norm(xref))
    plan.close()
