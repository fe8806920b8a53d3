"""The batch's own tiling: what Batch.tiling() reports after the bind, on
batches for which the library takes 8 rows and one for which it takes 4, gives
the bits of 4 rows with their chunks (the tiling never changes a result), and
stays as it is when set again."""
import pytest

from paper_1903_09043_amd import workloads as W

pytestmark = pytest.mark.gpu

SIZES = {"three_layers": [(64, 32)] * 3, "ragged": [(61, 7), (256, 128), (5, 3), (120, 30), (300, 64)],
         "many_small": [(20, 12)] * 700}
ROWS = {"three_layers": 8, "ragged": 8, "many_small": 4}


@pytest.mark.parametrize("name", SIZES)
def test_own_tiling(name):
    import torch
    import paper_1903_09043_amd as A
    cfgs = [W.rb(list(n), [2.0, 1.0], Ra=1e3)[0] for n in SIZES[name]]

    def run(tiling):
        B = A.Batch(cfgs)
        for k, c in enumerate(cfgs):
            if k < 8:
                U = A.Context(c).init_host(W.PROB_RB, [1.0, 0.5, -1.0, 1e-2], k)
                V = torch.as_tensor(U)
            B.view(k).copy_(V)
        if tiling:
            B.set_tiling(*tiling).bind()
        B.step(3)
        torch.cuda.synchronize()
        t, dt, cell, rc = B.read()
        assert rc == A.OK
        return B.tiling(), B.states.cpu(), t, dt

    own, U, t, dt = run(None)
    assert own[0] == ROWS[name]
    assert all(c["n"][1] % z == 0 for c, z in zip(cfgs, own[1]))
    for tiling in ((4, None), own):
        _, V, t2, dt2 = run(tiling)
        assert torch.equal(U, V) and (t == t2).all() and (dt == dt2).all()
    assert run(own)[0] == own
