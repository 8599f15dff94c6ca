"""Edge cases of the float64 engine's routes, against the per-baseline kernel
(variant 0, which never takes the engine) to the float64 bar, or bitwise against
the resident single-sky call where both run on the engine."""
import numpy as np
import pytest

from rime_synth import Observation
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
