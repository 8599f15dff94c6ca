"""Forward modes of the float32 256-thread kernel that stage the extended
sources' per-antenna terms from planes in HBM: bitwise equal to the kernel that
forms them itself (variant 1), whose arithmetic per term is the same, for skies
without point sources."""
import numpy as np
import pytest

from rime_synth import add_disks, make_problem, rngs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

R = pytest.importorskip("paper_1501_07719_amd")


# ragged 32-source tiles, 16-antenna blocks, channel pairs and channel blocks of
# the planes (16 channels, or 4 for planes of 1 MiB and more), above the
# smallest problem that takes planes (2^24 staged terms), and one below it
@pytest.mark.parametrize("na,ntime,nchan,ng,nx", [
    (17, 2, 5, 31, 33), (17, 60, 151, 31, 33), (33, 40, 95, 32, 0), (64, 21, 99, 33, 1),
    (50, 37, 51, 0, 65), (64, 5, 7, 2100, 0)])
def test_planes_equal_in_kernel_staging(na, ntime, nchan, ng, nx):
    pr = make_problem("c1", ntime=ntime, nchan=nchan, npsrc=0, ngsrc=ng, na=na, key=91)
    sky = R.DeviceSky.from_host(add_disks(pr.sky, nx, rngs(91)[5]))
    shape = (ntime, pr.obs.nbl, nchan, 4)
    plan = R.Plan(pr.obs)
    vis, chi = [], []
    for vi in (1, 5):
        assert R.rime_variant_info(R.MODE_CHI2, R.MIXED, vi) == (256, 2, 32)
        for mode in (R.MODE_PREDICT, R.MODE_CHI2):
            plan.set_variant(mode, R.MIXED, vi)
        ws = R.workspace(plan, R.MODE_CHI2, R.MIXED, 1, sky.nsrc)
        v = torch.full(shape, float("nan"), dtype=torch.complex64, device="cuda")
        R.rime_predict(plan, sky, R.MIXED, v, ws)
        vis.append(v)
        c = torch.empty(1, dtype=torch.float64, device="cuda")
        D = torch.as_tensor(pr.noise.astype(np.complex64), device="cuda")
        W = torch.as_tensor(pr.weight.astype(np.float32), device="cuda")
        R.rime_chi2(plan, sky, R.MIXED, D, W, c, ws)
        chi.append(c.item())
    torch.cuda.synchronize()
    assert torch.isfinite(torch.view_as_real(vis[0])).all()
    assert torch.equal(vis[0], vis[1])
    assert chi[0] == chi[1]
    plan.close()


# the gradient of the 256- and the 1024-thread kernel, whose adjoint also stages
# the beam-gradient factor
@pytest.mark.parametrize("off,on", [(2, 4), (1, 5)])
@pytest.mark.parametrize("na,ntime,nchan,ng,nx,beam", [
    (17, 2, 5, 31, 33, True), (17, 60, 151, 31, 33, True), (64, 21, 99, 33, 1, True),
    (50, 37, 51, 0, 65, False)])
def test_gradient_planes_equal_in_kernel_staging(off, on, na, ntime, nchan, ng, nx, beam):
    pr = make_problem("c1", ntime=ntime, nchan=nchan, npsrc=0, ngsrc=ng, na=na, key=92)
    if not beam:
        pr.obs.beam = False
    prec = R.MIXED
    sky = R.DeviceSky.from_host(add_disks(pr.sky, nx, rngs(92)[5]))
    D = torch.as_tensor(pr.noise.astype(np.complex64), device="cuda")
    W = torch.as_tensor(pr.weight.astype(np.float32), device="cuda")
    plan = R.Plan(pr.obs)
    out = []
    for vi in (off, on):
        assert R.rime_variant_info(R.MODE_CHI2_GRAD, prec, vi)[0] == (256 if vi in (1, 5) else 1024)
        plan.set_variant(R.MODE_CHI2_GRAD, prec, vi)
        ws = R.workspace(plan, R.MODE_CHI2_GRAD, prec, 1, sky.nsrc)
        c = torch.empty(1, dtype=torch.float64, device="cuda")
        g = torch.full((sky.nsrc, 10), float("nan"), dtype=torch.float64, device="cuda")
        R.rime_chi2_grad(plan, sky, prec, D, W, c, g, ws)
        out.append((c.item(), g))
    torch.cuda.synchronize()
    assert torch.isfinite(out[0][1]).all()
    assert out[0][0] == out[1][0]
    assert torch.equal(out[0][1], out[1][1])
    plan.close()
