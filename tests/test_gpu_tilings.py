"""Plans have the tile lists of every loop they may run from the start: calls on
fewer shots than warmed up with, and solves whose iterations take another tiling
than the first one, run under capture, where lists cannot be built."""
import numpy as np
import pytest
import torch

from tests.test_gpu_parity import _plan, _ragged_cfg

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def esi():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2211_06300_amd import esi as e
    e.load_library()
    return e


def test_graph_solve_with_separate_residual(esi):
    # iteration 0 runs short tiles, the captured ones 32-row tiles forward
    cfg = _ragged_cfg(nt=40)
    plan = _plan(esi, cfg)
    d = torch.randn(plan.data_shape(), generator=torch.Generator(device=DEV).manual_seed(3), device=DEV)
    plan.set_cg_rfuse(False)
    plan.set_cg_graph(True)
    x, work = plan.new_vec(3), torch.empty((3, *plan.vec_shape(3)), device=DEV)
    got = []
    for _ in range(3):
        _, rep = plan.cg_solve(d, max_iter=5, x=x, work=work)
        got.append((x.clone(), rep["res_hist"]))
        work[1].fill_(0.5)
        torch.cuda.synchronize()
    plan.set_cg_graph(False)
    ref, rep = plan.cg_solve(d, max_iter=5)
    for a, hist in got:
        assert torch.equal(a, ref)
        np.testing.assert_array_equal(hist, rep["res_hist"])
    plan.close()


def _line_plan(esi, ns, nt, stream=None, windows=False):
    """ns shots on 152 x 88 cells with a line of receivers: 24-row tiles for all
    of 60 shots (1500 workgroups of 16 rows), 8-row tiles for a few."""
    nx, nz, nb = 152, 88, 8
    rng = np.random.default_rng(2)
    src = np.stack([rng.integers(40, 100, ns), rng.integers(0, 12, ns)], 1).astype(np.int32)
    cols = np.arange(30, 130)
    rec = np.concatenate([np.stack([cols, np.full(cols.size, 3)], 1)] * ns).astype(np.int32)
    win = np.tile(np.array([[20, 140]], np.int32), (ns, 1)) if windows else None
    vel = torch.from_numpy(rng.uniform(1900.0, 2700.0, (nz, nx)).astype(np.float32)).to(DEV)
    return esi.Plan(ndim=2, nz=nz, nx=nx, nb=nb, nt=nt, dx=10.0, dt=1e-3, beta=1e-2, src=src,
                    rec_ptr=np.arange(ns + 1) * cols.size, rec=rec, vel=vel, stream=stream, window=win)


@pytest.mark.parametrize("windows", [False, True])
def test_captured_range_of_shots(esi, windows):
    ns, nt = 60, 9
    g = torch.Generator(device=DEV).manual_seed(4)
    w = torch.randn((ns, nt), generator=g, device=DEV)
    plain = _line_plan(esi, ns, nt, windows=windows)
    d = torch.randn(plain.data_shape(), generator=g, device=DEV)
    d1 = torch.randn(plain.data_shape(7, 1), generator=g, device=DEV)
    ref = plain.forward(w[7:8], shot0=7, nshots=1), plain.adjoint(d1, shot0=7, nshots=1)
    assert all(float(a.abs().max()) > 0 for a in ref)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        plan = _line_plan(esi, ns, nt, stream=stream, windows=windows)
        plan.forward(w)            # scratch for every shot
        plan.adjoint(d)
        out, mu = torch.empty_like(ref[0]), torch.empty_like(ref[1])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        plan.forward(w[7:8], shot0=7, nshots=1, out=out)
        plan.adjoint(d1, shot0=7, nshots=1, out=mu)
    for _ in range(3):
        out.fill_(float("nan"))
        mu.zero_()                 # (columns off the aperture are not written)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref[0]) and torch.equal(mu, ref[1])
        with torch.cuda.stream(stream):
            plan.forward(w)        # eager work between replays
        torch.cuda.synchronize()
    plan.close()
    plain.close()


def test_noalloc_takes_the_loops_own_tiling(esi):
    # a plan of 24-row tiles for all shots, called on one: 8-row tiles, two steps a launch
    ns, nt = 60, 9
    plan = _line_plan(esi, ns, nt)
    w = torch.randn((ns, nt), generator=torch.Generator(device=DEV).manual_seed(4), device=DEV)
    for n, rows in ((1, "8"), (30, "16"), (ns, "24")):
        plan.profile(True)
        out = plan.forward_noalloc(w[:n], nshots=n)
        ran = plan.profile_read()
        plan.profile(False)
        assert {k: v["launches"] for k, v in ran.items()} == {"SRC_POINT|GATHER": 1,
                                                             f"SRC_POINT|GATHER|TWO_STEP@56x{rows}": 4}
        assert torch.equal(out, plan.forward(w[:n], nshots=n))
    # a tiling that no call has built yet is refused, not replaced
    plan.set_launch_shape(4, 4)
    with pytest.raises(esi.EsiError, match="tile lists"):
        plan.forward_noalloc(w[:1], nshots=1)
    ref = plan.forward(w[:1], nshots=1)
    assert torch.equal(plan.forward_noalloc(w[:1], nshots=1), ref)
    plan.close()


def test_graph_solve_after_finer_tilings(esi):
    # other calls build tilings of more tiles than the solve's partials hold: the
    # captured iterations' partials stay where they are
    nx, nz, ns, nt = 801, 281, 8, 9
    rng = np.random.default_rng(5)
    src = np.stack([rng.integers(0, nx, ns), np.full(ns, 2)], 1).astype(np.int32)
    rec = np.concatenate([np.stack([np.arange(0, nx, 4), np.full(201, 3)], 1)] * ns).astype(np.int32)
    vel = torch.from_numpy(rng.uniform(1900.0, 2700.0, (nz, nx)).astype(np.float32)).to(DEV)
    plan = esi.Plan(ndim=2, nz=nz, nx=nx, nb=20, nt=nt, dx=10.0, dt=1e-3, beta=1e-2, src=src,
                    rec_ptr=np.arange(ns + 1) * 201, rec=rec, vel=vel)
    g = torch.Generator(device=DEV).manual_seed(4)
    w, d = torch.randn((ns, nt), generator=g, device=DEV), torch.randn(plan.data_shape(), generator=g, device=DEV)
    x, work = plan.new_vec(ns), torch.empty((3, *plan.vec_shape(ns)), device=DEV)
    plan.set_cg_graph(True)
    for other in (lambda: plan.forward(w[:1], nshots=1), lambda: plan.set_launch_shape(3, 3),
                  lambda: plan.normal_apply(x, out=work[2]), lambda: plan.set_time_block(2)):
        plan.cg_solve(d, max_iter=4, x=x, work=work)
        other()
        torch.cuda.synchronize()
    plan.set_cg_graph(False)
    ref, _ = plan.cg_solve(d, max_iter=4)
    plan.set_cg_graph(True)
    for _ in range(2):
        plan.cg_solve(d, max_iter=4, x=x, work=work)
        assert torch.equal(x, ref)
    plan.close()


@pytest.mark.parametrize("shape", [1, 2, 3, 4])
def test_graph_solve_with_separate_residual_on_set_shapes(esi, shape):
    cfg = _ragged_cfg(nt=30)
    plan = _plan(esi, cfg)
    d = torch.randn(plan.data_shape(), generator=torch.Generator(device=DEV).manual_seed(3), device=DEV)
    plan.set_cg_rfuse(False)
    plan.set_launch_shape(shape, shape)
    plan.set_cg_graph(True)
    got = [plan.cg_solve(d, max_iter=4)[0] for _ in range(2)]
    plan.set_cg_graph(False)
    ref, _ = plan.cg_solve(d, max_iter=4)
    assert all(torch.equal(x, ref) for x in got)
    plan.close()


@pytest.mark.parametrize("ns", [1, 30, 60, 130])
def test_autotuned_loops_run_what_was_timed(esi, ns):
    # the tiles that the reported choice stands for: its own, or for the default two
    # steps those of an untuned plan (8, 16, 24 and 32 rows here)
    nt = 9
    plan, plain = _line_plan(esi, ns, nt), _line_plan(esi, ns, nt)
    rows = {1: 6, 30: 5, 60: 3, 130: 2}[ns]
    p, Ap = plan.new_vec(ns), plan.new_vec(ns)

    def shapes(pl, n=ns):
        pl.profile(True)
        pl.normal_apply(p[:n], out=Ap[:n], nshots=n)
        ran = [v["flags"] for v in pl.profile_read().values()]
        pl.profile(False)
        return [max((f >> 16) & 7 for f in ran if bool(f & 8) == adj) or 1 for adj in (False, True)]

    assert shapes(plain) == [rows, rows]
    for probe in (False, True):
        ch = plan.autotune(p=None if probe else p, Ap=None if probe else Ap, probe=probe, force=True)
        assert shapes(plan) == [rows if c == 2 else c for c in ch]
        # the cached choice as well
        plan.set_time_block(2)
        assert plan.autotune(p=None if probe else p, Ap=None if probe else Ap, probe=probe) == ch
        assert shapes(plan) == [rows if c == 2 else c for c in ch]
        if ns > 1:   # a call on fewer shots takes shorter tiles, unless one step a launch was chosen
            assert shapes(plan, 1) == [1 if c == 1 else 6 for c in ch]
        plan.set_launch_shape(*ch)
        assert shapes(plan) == list(ch)
    plan.close()
    plain.close()


@pytest.mark.parametrize("ndim", [2, 3])
@pytest.mark.parametrize("steps", [1, 2])
def test_fixed_spread_equals_single_shots(esi, ndim, steps):
    # shots that repeat the receivers of the one before them, and shots that do not
    rng = np.random.default_rng(9)
    nx, nz, ny, nb, nt, ns = (70, 37, 1, 8, 20, 6) if ndim == 2 else (40, 20, 19, 4, 10, 6)
    dims = [nx, nz] + [ny] * (ndim - 2)
    spot = lambda n: np.stack([rng.integers(0, k, n) for k in dims], 1).astype(np.int32)
    a, b = spot(50), spot(9)
    a[11], a[12] = a[10], a[10]
    recs = [a, a, b, a, a, a[:0]]
    src = spot(ns)
    src[:, 1] = 2
    vel = torch.from_numpy(rng.uniform(1900.0, 2700.0, (nz, ny, nx) if ndim == 3 else (nz, nx)).astype(np.float32)).to(DEV)

    def plan_of(shots):
        pl = esi.Plan(ndim=ndim, nz=nz, ny=ny, nx=nx, nb=nb, nt=nt, dx=10.0, dt=1e-3, beta=1e-2, src=src[shots],
                      rec_ptr=np.concatenate([[0], np.cumsum([len(recs[s]) for s in shots])]),
                      rec=np.concatenate([recs[s] for s in shots]), vel=vel)
        pl.set_time_block(steps)
        return pl

    w = torch.randn((ns, nt), generator=torch.Generator(device=DEV).manual_seed(1), device=DEV)
    plan = plan_of(list(range(ns)))
    d = plan.forward(w)
    mu = plan.adjoint(d)
    at = 0
    for s in range(ns):
        one, n = plan_of([s]), nt * len(recs[s])
        assert torch.equal(one.forward(w[s:s + 1]), d[at:at + n]), s
        assert torch.equal(one.adjoint(d[at:at + n].clone()), mu[s:s + 1]), s
        at += n
        one.close()
    assert float(d.abs().max()) > 0 and float(mu.abs().max()) > 0
    plan.close()
