"""One-kernel adjoint step (2D, periodic x) on an MI355X.

Tiles of 12 x 12 cells with a 2-cell halo: grids of one cell row, of less
than a tile, of exactly one, of one cell more, and of several ragged tiles,
with every boundary, viscosity and low-Mach form the kernel takes; and the
forms next to them, which stay with the phase kernels.

(i)  against the oracle's brute-force reverse product (1e-10 of the largest
     entry, the bound of the phase kernels' own test);
(ii) against the phase kernels: the same chain-rule terms summed in another
     order (1e-12 of the largest entry, as for the 3D marches), into NaN-filled
     outputs and scratch, twice with the same bits.
"""
import numpy as np
import pytest

import oracle as O
from paper_1903_09043_amd import workloads as W
from tests import inputs as I
from tests.test_gpu_adjoint import perturbed, gpu_adjoint

pytestmark = pytest.mark.gpu

FORMS = ["walls", "walls_thetaoff_freeslip", "walls_inviscid", "strong_flow", "periodic_g0", "outflow_x"]


@pytest.fixture(scope="module")
def A():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1903_09043_amd as A
    A.lib()
    return A


def case(form, n):
    if form == "periodic_g0":
        cfg = dict(dim=2, n=n, L=[1.5, 0.8], gamma=1.4, g=0.0, mu=2e-3, kappa=3e-3, K=1.1, cfl=0.4, low_mach=1,
                   dt_mode=0, bc=[[0, 0], [0, 0]], wall_noslip=1, thermal=[0, 0], T_wall=[1.0, 1.0])
        return cfg, I.white_random(cfg, seed=61, amp=0.2)
    lm = 0 if form == "walls_thetaoff_freeslip" else 1
    cfg, prob, prm, seed = W.rb(n, [1.5, 1.0], Ra=1e4, seed=62, amp=1e-3, low_mach=lm)
    if form == "walls_thetaoff_freeslip":
        cfg = dict(cfg, wall_noslip=0, thermal=[1, 0])
    if form == "walls_inviscid":
        cfg = dict(cfg, mu=0.0, kappa=0.0)
    if form == "outflow_x":
        cfg = dict(cfg, bc=[[W.BC_OUTFLOW, W.BC_OUTFLOW], cfg["bc"][1]])
    return cfg, perturbed(cfg, prob, prm, seed, amp_u=0.3 if form == "strong_flow" else 0.05)


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("n", [[5, 6], [13, 5]], ids=str)
def test_vs_oracle(A, form, n):
    cfg, U = case(form, n)
    dt = O.dt(cfg, U)
    lam = np.random.default_rng(63).standard_normal(U.shape)
    g, pg = gpu_adjoint(A, cfg, U, lam, dt)
    o, gmu, gk = O.adjoint_dense(cfg, U, lam, dt)
    scale = np.abs(o).max()
    print(form, n, np.abs(g - o).max() / scale, pg, gmu, gk, flush=True)
    assert np.abs(g - o).max() <= 1e-10 * scale
    if cfg["mu"] > 0:
        assert abs(pg[0] - gmu) <= 1e-10 * max(abs(gmu), scale)
        assert abs(pg[1] - gk) <= 1e-10 * max(abs(gk), scale)


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("n", [[4, 8], [5, 5], [12, 12], [13, 25], [256, 6], [101, 67]], ids=str)
def test_vs_phase_kernels(A, form, n):
    import torch
    cfg, U = case(form, n)
    dt = torch.tensor([O.dt(cfg, U)], dtype=torch.float64)
    S = A.Solver(cfg)
    Ud = torch.as_tensor(U).cuda()
    lam = torch.as_tensor(np.random.default_rng(64).standard_normal(U.shape)).cuda()
    out = []
    for ref in (False, True, False):
        S.adjoint_workspace(ref).fill_(0xFF)
        pg = torch.tensor([0.5, -0.25], dtype=torch.float64, device="cuda")
        l0 = torch.full_like(lam, float("nan"))
        S.step_adjoint(Ud, lam, dt, lam_n=l0, param_grad=pg, ref=ref)
        torch.cuda.synchronize()
        out.append((l0.cpu().numpy(), pg.cpu().numpy()))
    (f, fp), (r, rp), (f2, fp2) = out
    scale = np.abs(r).max()
    print(form, n, np.abs(f - r).max() / scale, fp, rp, flush=True)
    assert np.abs(f - r).max() <= 1e-12 * scale
    assert np.abs(fp - rp).max() <= 1e-12 * max(np.abs(rp).max(), scale)
    assert np.array_equal(f, f2) and np.array_equal(fp, fp2)
