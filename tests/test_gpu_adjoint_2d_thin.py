"""One-kernel adjoint step (2D) on walled layers of one to four cell rows: at
one row a cell lies next to both walls and takes both ghosts' shares.  Against
the oracle and the phase kernels, with the bounds and the NaN-filled outputs
of the kernel's other sizes.  And an output that shares memory with the state,
for which the tiles (they write while others still read) are not taken: the
phase kernels' bits.
"""
import numpy as np
import pytest

import oracle as O
from tests.test_gpu_adjoint_2d import A, case, test_vs_oracle as vs_oracle, test_vs_phase_kernels as vs_phase  # noqa: F401

pytestmark = pytest.mark.gpu

FORMS = ["walls", "walls_thetaoff_freeslip", "walls_inviscid", "strong_flow"]


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("n", [[5, 1], [13, 2], [12, 3], [25, 4]], ids=str)
def test_thin(A, form, n):  # noqa: F811
    vs_oracle(A, form, n)
    vs_phase(A, form, n)


@pytest.mark.parametrize("shift", [0, 5, 13 * 25])
def test_output_over_state(A, shift):  # noqa: F811
    import torch
    cfg, U = case("walls", [13, 25])
    dt = torch.tensor([O.dt(cfg, U)], dtype=torch.float64)
    S = A.Solver(cfg)
    lam = torch.as_tensor(np.random.default_rng(65).standard_normal(U.shape)).cuda()
    out = []
    for ref in (False, True):
        buf = torch.empty(U.size + shift, dtype=torch.float64, device="cuda")
        buf[:U.size] = torch.as_tensor(U).reshape(-1).cuda()
        S.adjoint_workspace(ref).fill_(0xFF)
        pg = torch.zeros(2, dtype=torch.float64, device="cuda")
        l0 = buf[shift:].view(U.shape)
        S.step_adjoint(buf[:U.size].view(U.shape), lam, dt, lam_n=l0, param_grad=pg, ref=ref)
        out.append((l0.clone(), pg))
    (f, fp), (r, rp) = out
    assert torch.isfinite(f).all() and torch.equal(f, r) and torch.equal(fp, rp)
    apart = S.step_adjoint(torch.as_tensor(U).cuda(), lam, dt)  # the tiles
    assert (apart - f).abs().max() <= 1e-12 * f.abs().max()
