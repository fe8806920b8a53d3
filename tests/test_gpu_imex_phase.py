"""The passes around the conjugate-gradient solve of the implicit step
(csrc/ars_imex_phase.hip): sides of two and three cells, where a stencil meets
itself, rows past one block and past one XCD's run, with and without walls,
dissipation and the low-Mach correction, against the oracle's direct solve;
and several steps of one call (in place) against single calls, bit for bit.

The bound is the one of the other implicit tests: 1e-12 of each group of
variables, the residual being solved to 1e-13."""
import numpy as np
import pytest

import oracle as O
from tests import inputs as I
from tests import parity as PA

pytestmark = pytest.mark.gpu


def _cfg(n, walls, mu, lm):
    d = len(n)
    z = [1, 1] if walls else [0, 0]
    return dict(dim=d, n=list(n), L=[1.0, 0.8, 0.9][:d], gamma=1.4, g=0.5 if walls else 0.0, mu=mu, kappa=1.5 * mu,
                K=1.1, cfl=0.4, low_mach=lm, dt_mode=0, bc=[[0, 0]] * (d - 1) + [z], wall_noslip=1, thermal=[1, 0],
                T_wall=[1.0, 0.9])


@pytest.mark.parametrize("n", [(2, 2), (3, 2), (2, 131), (257, 3), (2, 2, 3), (3, 2, 2), (33, 2, 19)])
@pytest.mark.parametrize("walls,mu,lm", [(1, 2e-3, 1), (1, 0.0, 1), (0, 2e-3, 1), (1, 2e-3, 0)])
def test_vs_oracle(n, walls, mu, lm):
    import torch
    import paper_1903_09043_amd as A
    cfg = _cfg(n, walls, mu, lm)
    print(cfg["n"], walls, mu, lm, flush=True)
    U0 = I.smooth_random(cfg, seed=3)
    dt = O.dt(cfg, U0) * (3.0 if lm else 0.8)
    S, T = A.Solver(cfg), A.Solver(cfg)
    S.set_state(U0)
    T.set_state(U0)
    S.step_imex([dt] * 3)
    for _ in range(3):
        T.step_imex([dt])
    torch.cuda.synchronize()
    assert S.fault()[0] == 0
    assert torch.equal(S.U, T.U)
    r = O.run_imex(cfg, U0, 3, dt)
    assert r["status"] == 0
    assert PA.rel_err(cfg, S.numpy(), r["U"]) <= 1e-12
