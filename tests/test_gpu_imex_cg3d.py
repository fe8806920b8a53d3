"""3D conjugate-gradient solve of the implicit acoustic step at the edges of
its 32 x 16 columns of cells: one column, one cell more in each direction,
several columns, more planes than a unit takes, and the smallest sides,
walled and periodic, against the oracle's direct solve.

Tolerance: both solve the same system, the oracle to rounding and this to a
relative residual of 1e-12, so the pressures differ by at most cond * 1e-12 of
their norm a step.  The smallest eigenvalue is at least the diagonal
1/(rho c^2); at twice the explicit time step the largest is below 50 of it:
1e-10 over two steps.
"""
import pytest

import oracle as O
from paper_1903_09043_amd import workloads as W
from tests import inputs as I
from tests import parity as PA
from tests.test_gpu_adjoint import perturbed

pytestmark = pytest.mark.gpu

CASES = [("walls", [32, 16, 2]), ("walls", [33, 3, 8]), ("walls", [3, 17, 18]), ("walls", [5, 4, 45]),
         ("periodic", [34, 18, 2]), ("periodic", [2, 2, 150]), ("periodic", [66, 5, 3])]


@pytest.mark.parametrize("kind,n", CASES, ids=str)
def test_vs_oracle(kind, n):
    import torch
    import paper_1903_09043_amd as A
    if kind == "walls":
        cfg, prob, prm, seed = W.rb(n, [1.0, 1.0, 1.0], Ra=1e5, seed=81, amp=1e-2)
        U = perturbed(cfg, prob, prm, seed, amp_u=0.01)
    else:
        cfg = dict(dim=3, n=n, L=[1.0, 1.0, 1.0], gamma=1.4, g=0.0, mu=0.0, kappa=0.0, K=1.1, cfl=0.4, low_mach=1,
                   dt_mode=0, bc=[[0, 0]] * 3, wall_noslip=1, thermal=[0, 0], T_wall=[1.0, 1.0])
        U = I.smooth_random(cfg, 82, amp_u=0.05, modes=3)
    dt = 2.0 * O.dt(cfg, U)
    S = A.Solver(cfg)
    S.set_state(U)
    its = S.step_imex([dt] * 2, tol=1e-12)
    torch.cuda.synchronize()
    r = O.run_imex(cfg, U, 2, dt)
    assert r["status"] == 0
    err = PA.rel_err(cfg, S.numpy(), r["U"])
    print(kind, n, "iterations", its, "error", err, flush=True)
    assert its > 0
    assert err <= 1e-10
