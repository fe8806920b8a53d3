"""The preconditioned implicit step in 3D where the y transform takes several
tiles of mirror pairs in every batch: state, bound and iteration count of the
other sizes."""
import pytest

from tests.test_gpu_imex_trig import test_trig_preconditioned_step as step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,walls", [((34, 66, 2), False), ((3, 67, 12), True)])
def test_several_tiles(n, walls):
    step(n, walls)
