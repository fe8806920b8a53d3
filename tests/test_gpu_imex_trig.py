"""The implicit acoustic step with the trigonometric preconditioner, on
low-Mach states whose coefficients are nearly constant (where it is chosen),
against the oracle's direct solve: sides that are one product tile, one more
and one less, several ragged tiles and stages, shorter than a stage, periodic
and walled, in 2D and 3D.  Tolerance: the solve ends at a relative residual
of 1e-13, so Pi is known to 1e-13 times the operator's condition number,
1 + sum nu_d^2 with nu_d = dt c / dx_d, and the momentum to nu / gamma times
that on the scale of rho c, per step (the plain solver is as far from the
oracle on these states).
"""
import numpy as np
import pytest

import oracle as O
from tests import inputs as I
from tests import parity as PA

pytestmark = pytest.mark.gpu

SIZES = [((64, 64), False), ((65, 63), False), ((33, 130), False), ((128, 40), True), ((40, 97), True),
         ((64, 65), True), ((5, 6, 34), False), ((7, 5, 33), True)]


@pytest.mark.parametrize("n,walls", SIZES, ids=["%s%s" % ("x".join(map(str, n)), "-walls" * w) for n, w in SIZES])
def test_trig_preconditioned_step(n, walls):
    import torch
    import paper_1903_09043_amd as A
    D, Ma = len(n), 1e-2
    cfg = dict(dim=D, n=list(n), L=[1.0, 0.8, 0.9][:D], gamma=1.4, g=1.0 if walls else 0.0, mu=1e-3, kappa=1e-3,
               K=1.1, cfl=0.4, low_mach=1, dt_mode=0, bc=[[0, 0]] * (D - 1) + [[1, 1] if walls else [0, 0]],
               wall_noslip=1, thermal=[0, 0], T_wall=[1.0, 1.0])
    U0 = I.smooth_random(cfg, seed=5, p0=1.0 / (1.4 * Ma * Ma), amp_rho=1e-3, amp_u=0.5, amp_p=Ma * Ma)
    dt = O.dt(cfg, U0) * 30.0
    S = A.Solver(cfg).set_state(U0)
    its = S.step_imex([dt] * 2)
    torch.cuda.synchronize()
    assert S.fault()[0] == 0
    r = O.run_imex(cfg, U0, 2, dt)
    assert r["status"] == 0
    err = PA.rel_err(cfg, S.numpy(), r["U"])
    print("iterations", its, "parity", err, flush=True)
    nu = [dt / Ma * n[a] / cfg["L"][a] for a in range(D)]
    assert err <= 2 * 1e-13 * (1.0 + sum(v * v for v in nu)) * max(nu) / 1.4
    assert its <= 20  # plain conjugate gradients need some 50 a step at acoustic CFL 30
