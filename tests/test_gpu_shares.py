"""Shares of the (tile, plane) pairs: grids whose tiles get one chunk, several
equal ones, several with a shorter last one, one plane each, and grids with
more tiles than workgroups (shares across tiles), for the fused step and the
three adjoint marches, against the phase-kernel paths.  Tolerances: the step's
two paths share their expressions (a few ulp of the largest value); the
adjoint's differ in the order of their sums (1e-12 of the largest entry, as
in the marches' own tests).
"""
import pytest

from paper_1903_09043_amd import workloads as W
from tests import inputs as I

pytestmark = pytest.mark.gpu

GRIDS = [[32, 10, 1], [33, 11, 7], [40, 24, 64], [64, 40, 67], [101, 20, 131], [640, 140, 3], [64, 60, 5]]


def _setup(n):
    import torch
    import paper_1903_09043_amd as A
    cfg = W.rb(n, [1.0] * len(n), Ra=1e4)[0]
    U = A.Context(cfg).init_host(W.PROB_RB, [1.0, 0.5, -1.0, 1e-2], 3)
    V = I.smooth_random(cfg, 7, amp_u=0.05)
    for k in range(len(n)):
        U[1 + k] = U[0] * V[1 + k] / V[0]
    U[-1] += 0.5 * (U[1:-1] ** 2).sum(0) / U[0]
    return torch, A.Solver(cfg).set_state(U)


@pytest.mark.parametrize("n", GRIDS + [[64, 33], [61, 1], [1300, 700], [60, 5000]], ids=lambda n: "x".join(map(str, n)))
def test_step_shares(n):
    torch, S = _setup(n)
    U0, d = S.U.clone(), S.dt.repeat(2).contiguous()
    S.step_sched(d)
    a = S.U.clone()
    S.U.copy_(U0)
    S.step_ref(d)
    for v in range(a.shape[0]):
        assert (a[v] - S.U[v]).abs().max() <= 1e-15 * S.U[-1].abs().max()


@pytest.mark.parametrize("n", GRIDS[1:], ids=lambda n: "x".join(map(str, n)))
def test_adjoint_shares(n):
    torch, S = _setup(n)
    g = torch.Generator(device="cpu").manual_seed(3)
    lam = torch.randn(S.U.shape, generator=g, dtype=torch.float64).cuda()
    out = []
    for ref in (False, True):
        pg = torch.zeros(2, dtype=torch.float64, device="cuda")
        out.append((S.step_adjoint(S.U, lam, S.dt, param_grad=pg, ref=ref), pg))
    (a, pa), (b, pb) = out
    assert (a - b).abs().max() <= 1e-12 * b.abs().max()
    # the parameter sums: n random terms of either sign
    assert (pa - pb).abs().max() <= 1e-12 * pb.abs().max() * a.numel() ** 0.5
