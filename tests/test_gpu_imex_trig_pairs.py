"""The trigonometric preconditioner's half products at the edges of their
32-pair tiles and 16-deep stages, where a length's mirror pairs leave a single
middle (or, with cosine modes, a missing last odd mode): state, bound and
iteration count of the preconditioned step's other sizes."""
import pytest

from tests.test_gpu_imex_trig import test_trig_preconditioned_step as step

pytestmark = pytest.mark.gpu


# pairs: cas n / 2 + 1, cos (n + 1) / 2
@pytest.mark.parametrize("n,walls", [((62, 31), False), ((30, 61), False), ((34, 66), False), ((62, 63), True),
                                     ((63, 33), True), ((94, 31), True)])
def test_pairs(n, walls):
    step(n, walls)
