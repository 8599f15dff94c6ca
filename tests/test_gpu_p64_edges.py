"""Edge cases of the float64 engine's routes, against the per-baseline kernel
(variant 0, which never takes the engine) to the float64 bar, or bitwise against
the resident single-sky call where both run on the engine."""
import numpy as np
import pytest

from rime_synth import Observation, make_problem, random_die, stokes_per_time
from tests._helpers import TOL, grad_errors, rel
from tests.test_gpu_p64 import problem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

R = pytest.importorskip("paper_1501_07719_amd")
F64 = dict(dtype=torch.float64, device="cuda")


def dev(D, W, prec=0):
    if prec != R.FP64:
        D, W = D.astype(np.complex64), W.astype(np.float32)
    return torch.as_tensor(D, device="cuda"), torch.as_tensor(W, device="cuda")


def gradient(obs, sky, D, W, variant=1, fill=0xFF, prec=0, ws_bytes=None):
    """chi^2 and gradient of one sky, over a workspace of `fill` bytes."""
    plan = R.Plan(obs)
    if prec == R.FP64:
        plan.set_variant(R.MODE_CHI2_GRAD, prec, variant)
    Dd, Wd = dev(D, W, prec)
    n = ws_bytes or plan.workspace_size(R.MODE_CHI2_GRAD, prec, 1, sky.nsrc)
    ws = torch.full((n,), fill, dtype=torch.uint8, device="cuda")
    chi2, grad = torch.empty(1, **F64), torch.full((sky.nsrc, 10), float("nan"), **F64)
    R.rime_chi2_grad(plan, R.DeviceSky.from_host(sky), prec, Dd, Wd, chi2, grad, ws)
    torch.cuda.synchronize()
    plan.close()
    return chi2.item(), grad.cpu().numpy()


def check(a, b, sky):
    assert np.isfinite(a[1]).all()
    assert rel(a[0], b[0]) <= TOL[0]
    errs = grad_errors(a[1], b[1], sky.npsrc)
    assert max(errs.values()) <= TOL[0], errs


@pytest.mark.parametrize("npsrc,ng,nx", [(33, 0, 0), (0, 49, 0), (65, 0, 35), (32, 33, 0)])
def test_gradient_without_beam_ignores_the_workspace(npsrc, ng, nx):
    """Source counts that leave padding in the planes' rows (33, 49, 100, 65 of
    40, 56, 104, 72): what the workspace held before must not reach the sums."""
    obs, sky, D, W = problem(17, 2, 3, npsrc, ng, nx, "", beam=False)
    check(gradient(obs, sky, D, W), gradient(obs, sky, D, W, 0), sky)


@pytest.mark.parametrize("beam", [True, False])
@pytest.mark.parametrize("dead", [[5], [3, 16], [0, 17, 32]])
def test_antennas_without_baselines(dead, beam):
    """An antenna that no baseline holds may have undefined coordinates and
    pointing: the gradient must not depend on them."""
    obs, sky, D, W = problem(33, 2, 3, 40, 36, 0, "", beam=beam)
    keep = ~(np.isin(obs.ant1, dead) | np.isin(obs.ant2, dead))
    uvw = obs.uvw.copy()
    uvw[:, dead] = np.nan
    pnt = None if obs.pointing is None else obs.pointing.copy()
    if pnt is not None:
        pnt[:, dead] = np.nan
    obs = Observation(**{**obs.__dict__, "ant1": obs.ant1[keep], "ant2": obs.ant2[keep],
                         "uvw": uvw, "pointing": pnt})
    D, W = np.ascontiguousarray(D[:, keep]), np.ascontiguousarray(W[:, keep])
    check(gradient(obs, sky, D, W), gradient(obs, sky, D, W, 0), sky)


@pytest.mark.parametrize("prec", [0, 1, 2])
def test_dropped_antennas_are_not_read(prec):
    """Undefined coordinates of antennas without baselines give the bits that any
    others give, in every precision."""
    obs, sky, D, W = problem(40, 2, 4, 70, 40, 20, "")
    dead = [2, 31, 39]
    keep = ~(np.isin(obs.ant1, dead) | np.isin(obs.ant2, dead))
    D, W = np.ascontiguousarray(D[:, keep]), np.ascontiguousarray(W[:, keep])
    out = []
    for x in (1.0, np.nan):
        uvw, pnt = obs.uvw.copy(), obs.pointing.copy()
        uvw[:, dead] *= x
        pnt[:, dead] *= x
        o = Observation(**{**obs.__dict__, "ant1": obs.ant1[keep], "ant2": obs.ant2[keep],
                           "uvw": uvw, "pointing": pnt})
        out.append(gradient(o, sky, D, W, prec=prec))
    assert np.isfinite(out[0][1]).all() and out[0][0] == out[1][0]
    np.testing.assert_array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("ng", [0, 40])
def test_common_offset_of_the_antenna_coordinates(ng):
    """Only coordinate differences enter the model; antennas given from the
    Earth's centre (6.4e6 m) instead of the array's keep the gradient's
    accuracy.  The baselines are as in the centred array to 6.4e6 2^-53 =
    7e-10 m, and both kernels see the same ones."""
    obs, sky, D, W = problem(20, 2, 4, 64, ng, 0, "")
    uvw = obs.uvw * 0.05 + np.array([6.4e6, -3.1e6, 2.2e6])
    obs = Observation(**{**obs.__dict__, "uvw": uvw})
    check(gradient(obs, sky, D, W), gradient(obs, sky, D, W, 0), sky)


@pytest.mark.parametrize("prec", [0, 2])
@pytest.mark.parametrize("graph", [False, True])
def test_batch_of_one_set(prec, graph):
    obs, sky, D, W = problem(20, 2, 5, 40, 30, 10, "")
    plan = R.Plan(obs)
    Dd, Wd = dev(D, W, prec)
    ds = R.DeviceSky.from_host(sky)
    batch = R.Batch(plan, [ds])
    got, ref = [], []
    with torch.cuda.stream(torch.cuda.Stream()):
        for mode in (R.MODE_CHI2, R.MODE_CHI2_GRAD):
            for vi in range(R.rime_variant_count(mode, prec)):
                plan.set_variant(mode, prec, vi)
                chi2, grad = torch.full((1,), -1.0, **F64), torch.full((sky.nsrc, 10), -1.0, **F64)
                g = grad if mode == R.MODE_CHI2_GRAD else None
                ws = torch.empty(batch.workspace_size(mode, prec), dtype=torch.uint8,
                                 device="cuda")
                for _ in range(2):
                    R.rime_chi2_batched(batch, prec, Dd, Wd, chi2, g, ws, use_graph=graph)
                torch.cuda.current_stream().synchronize()
                got.append((chi2.item(), grad.cpu().numpy()))
                chi2, grad = torch.full((1,), -1.0, **F64), torch.full((sky.nsrc, 10), -1.0, **F64)
                ws = R.workspace(plan, mode, prec, 1, sky.nsrc)
                if mode == R.MODE_CHI2:
                    R.rime_chi2(plan, ds, prec, Dd, Wd, chi2, ws)
                else:
                    R.rime_chi2_grad(plan, ds, prec, Dd, Wd, chi2, grad, ws)
                torch.cuda.current_stream().synchronize()
                ref.append((chi2.item(), grad.cpu().numpy()))
    for a, b in zip(got, ref):
        assert a[0] == b[0]
        np.testing.assert_array_equal(a[1], b[1])
    batch.close()
    plan.close()


def test_many_uneven_sets_in_one_batch():
    """Sums of a batch whose (largest set) x (chunks) x (sets) launch is past 2^24
    workgroups: 65100 sets of one source and one of 6600."""
    obs, sky, D, W = problem(3, 1, 64, 6600, 0, 0, "")
    big, one = R.DeviceSky.from_host(sky), R.DeviceSky.from_host(sky.subset(1, 0))
    n = 65100
    plan = R.Plan(obs)
    batch = R.Batch(plan, [one] * n + [big])
    Dd, Wd = dev(D, W)
    ws = torch.empty(batch.workspace_size(R.MODE_CHI2_GRAD, 0), dtype=torch.uint8, device="cuda")
    chi2 = torch.full((n + 1,), -1.0, **F64)
    grad = torch.full((batch.total_src, 10), float("nan"), **F64)
    R.rime_chi2_batched(batch, 0, Dd, Wd, chi2, grad, ws)
    torch.cuda.synchronize()
    c, g = chi2.cpu().numpy(), grad.cpu().numpy()
    ref = [gradient(obs, s, D, W) for s in (sky.subset(1, 0), sky)]
    assert (c[:n] == c[0]).all() and (g[:n] == g[0]).all()
    check((c[0], g[:1]), ref[0], sky.subset(1, 0))
    check((c[n], g[n:]), ref[1], sky)
    batch.close()
    plan.close()


def engine_sizes(na, ntime, nchan, counts, prec, mode):
    obs = make_problem("c1", ntime=ntime, nchan=nchan, npsrc=4, ngsrc=0, na=na, key=95,
                       dense=False).obs
    plan = R.Plan(obs)
    out = [plan.workspace_size(mode, prec, 1, n) for n in counts]
    plan.close()
    return out


@pytest.mark.parametrize("mode,prec", [(0, 0), (1, 0), (2, 0), (1, 2), (2, 2)])
@pytest.mark.parametrize("na,ntime,nchan", [(64, 1, 64), (20, 7, 5), (64, 3, 17), (33, 50, 3)])
def test_workspace_grows_with_the_sky(mode, prec, na, ntime, nchan):
    """A workspace for the largest sky holds what smaller ones take."""
    counts = [1, 31, 32, 33, 63, 64, 65, 100, 128, 192, 193, 250, 256, 300, 500, 511, 512, 700,
              1000, 2000, 5000]
    sizes = engine_sizes(na, ntime, nchan, counts, prec, mode)
    assert all(a <= b for a, b in zip(sizes, sizes[1:])), list(zip(counts, sizes))


def test_ragged_streamed_chunk_runs_on_the_engine():
    """64 antennas, 64 channels: a chunk of two timesteps takes fewer partial
    sums than the last chunk of one.  Streamed sums equal those of the two
    resident calls bit by bit."""
    obs, sky, D, W = problem(64, 3, 64, 64, 36, 0, "")
    plan = R.Plan(obs)
    n = R.rime_streamed_workspace_size(plan, R.MODE_CHI2_GRAD, 0, sky.nsrc, 2)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    chi2, grad = torch.empty(1, **F64), torch.empty((sky.nsrc, 10), **F64)
    R.rime_chi2_streamed(plan, R.DeviceSky.from_host(sky), 0, torch.as_tensor(D).pin_memory(),
                         torch.as_tensor(W).pin_memory(), chi2, grad, 2, ws)
    torch.cuda.synchronize()
    plan.close()
    a, b = (gradient(obs.time_slice(t0, t1), sky, np.ascontiguousarray(D[t0:t1]),
                     np.ascontiguousarray(W[t0:t1])) for t0, t1 in ((0, 2), (2, 3)))
    assert chi2.item() == a[0] + b[0]
    np.testing.assert_array_equal(grad.cpu().numpy(), a[1] + b[1])


@pytest.mark.parametrize("prec", [0, 2])
def test_smaller_skies_in_a_workspace_for_the_largest(prec):
    """A workspace and batch lanes sized by the largest sky run the smaller ones
    on the same kernels as a workspace of their own: results bit by bit."""
    obs, sky, D, W = problem(64, 1, 64, 256, 256, 0, "")
    skies = [sky.subset(a, b) for a, b in ((256, 256), (192, 192), (64, 64), (50, 40))]
    plan = R.Plan(obs)
    n = plan.workspace_size(R.MODE_CHI2_GRAD, prec, 1, skies[0].nsrc)
    own = [gradient(obs, s, D, W, prec=prec) for s in skies]
    for s, b in zip(skies, own):
        a = gradient(obs, s, D, W, prec=prec, ws_bytes=n)
        assert a[0] == b[0]
        np.testing.assert_array_equal(a[1], b[1])
    Dd, Wd = dev(D, W, prec)
    batch = R.Batch(plan, [R.DeviceSky.from_host(s) for s in skies])
    ws = torch.empty(batch.workspace_size(R.MODE_CHI2_GRAD, prec), dtype=torch.uint8,
                     device="cuda")
    chi2 = torch.empty(len(skies), **F64)
    grad = torch.empty((batch.total_src, 10), **F64)
    R.rime_chi2_batched(batch, prec, Dd, Wd, chi2, grad, ws)
    torch.cuda.synchronize()
    g, at = grad.cpu().numpy(), 0
    for i, (s, b) in enumerate(zip(skies, own)):
        assert chi2[i].item() == b[0]
        np.testing.assert_array_equal(g[at:at + s.nsrc], b[1])
        at += s.nsrc
    batch.close()
    plan.close()


def test_main_events_of_a_batch_by_sets():
    """The main-event hooks bracket the engine's kernels of a batched call that
    runs set by set: most of what the timing events bracket."""
    obs, sky, D, W = problem(64, 12, 45, 64, 64, 0, "")
    plan = R.Plan(obs)
    batch = R.Batch(plan, [R.DeviceSky.from_host(sky) for _ in range(4)])
    Dd, Wd = dev(D, W)
    ws = torch.empty(batch.workspace_size(R.MODE_CHI2_GRAD, 0), dtype=torch.uint8, device="cuda")
    chi2, grad = torch.empty(4, **F64), torch.empty((batch.total_src, 10), **F64)
    R.rime_chi2_batched(batch, 0, Dd, Wd, chi2, grad, ws)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    for e in ev:
        e.record()
    torch.cuda.synchronize()
    plan.set_timing_events(ev[0], ev[1])
    plan.set_main_events(ev[2], ev[3])
    R.rime_chi2_batched(batch, 0, Dd, Wd, chi2, grad, ws)
    torch.cuda.synchronize()
    plan.set_timing_events(None, None)
    plan.set_main_events(None, None)
    assert ev[2].elapsed_time(ev[3]) >= 0.5 * ev[0].elapsed_time(ev[1]) > 0.0
    batch.close()
    plan.close()


def smallest_workspace(call, full):
    """Least bytes that `call(ws)` accepts."""
    lo, hi = 0, full  # refused, accepted
    while hi - lo > 256:
        mid = (lo + hi) // 512 * 256
        try:
            call(torch.empty(mid, dtype=torch.uint8, device="cuda"))
            hi = mid
        except R.RimeError as e:
            assert e.status == 2
            lo = mid
    return hi


@pytest.mark.parametrize("na,ntime,nchan,npsrc,ng,engine", [
    (15, 1, 2, 32, 0, True), (33, 3, 4, 64, 40, True), (64, 9, 9, 33, 41, True),
    (64, 9, 9, 33, 30, False),
    (15, 1, 2, 31, 0, False), (14, 2, 2, 64, 0, False)])
def test_route_of_the_gradient(na, ntime, nchan, npsrc, ng, engine):
    """The engine's sums and the per-baseline kernel's differ in their last bits:
    a call with the least workspace it accepts (never the engine) gives other
    bits exactly when the full workspace takes the engine.  From 32 sources on,
    lanes half full, over more than 96 baselines."""
    obs, sky, D, W = problem(na, ntime, nchan, npsrc, ng, 0, "")
    plan = R.Plan(obs)
    ds, (Dd, Wd) = R.DeviceSky.from_host(sky), dev(D, W)
    chi2, grad = torch.empty(1, **F64), torch.empty((sky.nsrc, 10), **F64)
    call = lambda ws: R.rime_chi2_grad(plan, ds, 0, Dd, Wd, chi2, grad, ws)  # noqa: E731
    full = plan.workspace_size(R.MODE_CHI2_GRAD, 0, 1, sky.nsrc)
    least = smallest_workspace(call, full)
    out = []
    for n in (full, least):
        call(torch.empty(n, dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        out.append((chi2.item(), grad.cpu().numpy()))
    plan.close()
    check(*out, sky)
    assert np.array_equal(out[0][1], out[1][1]) != engine


@pytest.mark.parametrize("prec", [0, 2])
@pytest.mark.parametrize("terms", [False, True])
def test_passes_over_time_and_channel_groups(prec, terms):
    """1400 sources over 64 antennas, 64 channels and 17 timesteps: two passes
    over time (9 and 8 timesteps), several channels per adjoint item; against
    the per-baseline kernel (float64-residual: the forward variant)."""
    obs, sky, D, W = problem(64, 17, 64, 700, 500, 200, "")
    rng = np.random.default_rng(6)
    extra = {}
    if terms:
        extra = dict(die=torch.as_tensor(random_die(17, 64, 64, rng), device="cuda"),
                     stokes_t=torch.as_tensor(stokes_per_time(sky, 17, rng), device="cuda"))
    Dd, Wd = dev(D, W, prec)
    ds = R.DeviceSky.from_host(sky)
    out = []
    for vi in (1, 0):
        plan = R.Plan(obs)
        plan.set_variant(R.MODE_CHI2_GRAD if prec == 0 else R.MODE_CHI2, prec, vi)
        chi2, grad = torch.empty(1, **F64), torch.full((sky.nsrc, 10), float("nan"), **F64)
        g = {f"grad_{k}": torch.full_like(v, float("nan")) for k, v in extra.items()}
        n = R.rime_workspace_size_ex(plan, R.MODE_CHI2_GRAD, prec, sky.nsrc,
                                     **{k: True for k in (*extra, *g)})
        ws = torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda")
        R.rime_chi2_ex(plan, ds, prec, Dd, Wd, chi2, grad, ws, **extra, **g)
        torch.cuda.synchronize()
        out.append((chi2.item(), grad.cpu().numpy(), {k: v.cpu().numpy() for k, v in g.items()}))
        plan.close()
    a, b = out
    # (the adjoint of the float64-residual mode is float32 in both)
    tol = TOL[prec]
    assert rel(a[0], b[0]) <= TOL[0]
    assert max(grad_errors(a[1], b[1], sky.npsrc).values()) <= tol
    for k in a[2]:
        assert np.linalg.norm(a[2][k] - b[2][k]) <= tol * np.linalg.norm(b[2][k]), k


def test_workspace_of_the_engine_is_bounded():
    """64 antennas, 100 timesteps, 64 channels, 1500 sources, gradient: planes
    of all timesteps take 15 GB; a call asks for one pass over time."""
    n, = engine_sizes(64, 100, 64, [1500], 0, R.MODE_CHI2_GRAD)
    assert n <= 3 << 30


@pytest.mark.parametrize("na,ntime,nchan,prec,n", [
    (20, 3, 8, 1, 1811), (16, 5, 8, 1, 1047), (27, 5, 7, 2, 1194), (32, 1, 2, 2, 18272)])
def test_largest_sky_of_the_fixed_workspace(na, ntime, nchan, prec, n):
    """The float32 planes are packed: the most point sources that the library's
    32 MiB hold beside the other regions."""
    obs = make_problem("c1", ntime=ntime, nchan=nchan, npsrc=4, ngsrc=0, na=na, key=1,
                       dense=False).obs
    plan = R.Plan(obs)
    shape = (ntime, plan.nbl, nchan, 4)
    D = torch.zeros(shape, dtype=torch.complex64, device="cuda")
    W = torch.ones(shape, dtype=torch.float32, device="cuda")
    for k, fits in ((n, True), (2 * n, False)):
        sky = R.DeviceSky(lm=torch.zeros((k, 2), **F64), stokes=torch.ones((k, 4), **F64),
                          alpha=torch.zeros(k, **F64), gshape=torch.zeros((0, 3), **F64),
                          npsrc=k, ngsrc=0)
        chi2, grad = torch.empty(1, **F64), torch.full((k, 10), float("nan"), **F64)
        if fits:
            R.rime_chi2_grad_noalloc(plan, sky, prec, D, W, chi2, grad)
            torch.cuda.synchronize()
            assert torch.isfinite(grad).all()
        else:
            with pytest.raises(R.RimeError):
                R.rime_chi2_grad_noalloc(plan, sky, prec, D, W, chi2, grad)
    plan.close()
