"""The tile heights that plans choose by themselves, at shot counts that land on
each of them: every entry point against one-step launches, bit for bit, with the
height that ran taken from the profile."""
import pytest
import torch

from tests.test_gpu_tiles2d import _everything, _plan

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def esi():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2211_06300_amd import esi as e
    e.load_library()
    return e


# the variants below that have every height; others run on 32 rows
HEIGHTS = {"SRC_POINT|GATHER", "SRC_DENSE|GATHER", "INJ|OUT", "INJ|NORMAL", "SRC_DENSE|PENALTY", "SRC_POINT|STORE",
           "INJ|CORR", "SRC_DENSE|GATHER|RUPD", "CG_FUSE|GATHER|RUPD", "INJ|NORMAL|RUPD"}


def _all(esi, plan, nt, ns):
    out, x = _everything(esi, plan, nt, ns)
    g = torch.Generator(device=DEV).manual_seed(6)
    w, d = torch.randn((ns, nt), generator=g, device=DEV), torch.randn(plan.data_shape(), generator=g, device=DEV)
    return out + [plan.gradient(esi.GRAD_SEED, w, d, kind=esi.SRC_POINT, ckpt_every=5)], x


# workgroups of (8, 16, 24) rows a shot: 39, 21, 15; 56, 28, 20; 10, 5, 4
@pytest.mark.parametrize("grid,ns,rows", [
    ((152, 88, 8), 19, "8"), ((152, 88, 8), 20, "16"), ((152, 88, 8), 48, "16"), ((152, 88, 8), 49, "24"),
    ((152, 88, 8), 85, "24"), ((152, 88, 8), 86, "32"), ((153, 89, 8), 30, "16"), ((153, 89, 8), 60, "24"),
    ((37, 70, 4), 100, "16"), ((37, 70, 4), 230, "24")])
def test_own_heights_bitwise(esi, grid, ns, rows):
    nt = 7
    plan = _plan(esi, *grid, ns, nt, 40)
    plan.set_time_block(1)
    ref, xref = _all(esi, plan, nt, ns)
    plan.set_time_block(2)
    plan.profile(True)
    got, x = _all(esi, plan, nt, ns)
    ran = {k.split("|TWO_STEP@")[0]: k.split("@56x")[1] for k in plan.profile_read() if "TWO_STEP" in k}
    plan.profile(False)
    assert set(ran) >= HEIGHTS, HEIGHTS - set(ran)
    assert {k: v for k, v in ran.items() if k in HEIGHTS} == dict.fromkeys(HEIGHTS, rows)
    assert all(v == "32" for k, v in ran.items() if k not in HEIGHTS), ran
    for k, (a, b) in enumerate(zip(ref, got)):
        assert torch.equal(a, b), k
    # float64 partials over other tiles: as in test_gpu_tiles2d
    assert float(torch.linalg.norm(x - xref)) <= 3 * 2 ** -23 * 4 * float(torch.linalg.norm(xref))
    plan.close()
