"""Dense plane spectra about the longest row whose w the transform forms in LDS
(455 cells; one more takes the separate pass), and planes of fewer than 16
rows, against numpy's FFT: the shells' sums agree to rounding, whose bound is
1e-12 of the plane's energy as for the other sizes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(455, 17), (456, 17), (100, 15), (127, 33), (3, 5)])
def test_against_numpy(nx, ny):
    import torch
    import paper_1903_09043_amd as A
    cfg = dict(dim=3, n=[nx, ny, 3], L=[1.0, 1.0, 1.0], gamma=1.4, g=0.0, mu=0.0, kappa=0.0, K=1.1, cfl=0.4,
               low_mach=1, dt_mode=0, bc=[[0, 0]] * 3, wall_noslip=1, thermal=[0, 0], T_wall=[1.0, 1.0])
    rng = np.random.default_rng(9)
    U = rng.standard_normal((5, 3, ny, nx))
    U[0] = 1.0 + 0.2 * rng.random(U[0].shape)
    U[4] += 50.0
    S = A.Solver(cfg).set_state(U)
    E = np.asarray(torch.as_tensor(S.spectrum()).cpu())
    w = U[1:4, 1] / np.sqrt(U[0, 1])
    P = (np.abs(np.fft.fft2(w)) ** 2).sum(0) / (2.0 * (nx * ny) ** 2)
    k = np.sqrt(np.fft.fftfreq(ny, 1.0 / ny)[:, None] ** 2 + np.fft.fftfreq(nx, 1.0 / nx)[None, :] ** 2)
    ref = np.bincount(np.rint(k).astype(int).ravel(), P.ravel(), minlength=len(E))
    assert len(E) == len(ref)
    assert np.abs(E - ref).max() <= 1e-12 * ref.sum()
