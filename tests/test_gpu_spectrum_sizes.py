"""Plane spectrum at the edges of its two transforms, against the oracle's
spectrum with the bound derived in tests/test_gpu_spectrum.py: FFT sides of
one to 2048 cells (odd and even numbers of radix-2 stages, one and all
components at a time, fewer rows than a block takes) and dense sides around
the 16-wide matrix tiles and the 64-wide groups of half-plane columns.
"""
import pytest

import oracle as O
from tests import inputs as I
from tests.test_gpu_spectrum import A, cfg_of, check, gpu_spectrum  # noqa: F401

pytestmark = pytest.mark.gpu

FFT = [[1, 1], [1, 8], [2, 2], [4, 1], [8, 4], [4, 16], [128, 2], [256, 256], [512, 64], [1024, 8], [2048, 4],
       [4, 1024], [2, 2048]]
DENSE = [[3, 1], [1, 3], [2, 3], [3, 2], [15, 17], [33, 16], [64, 65], [126, 31], [128, 33], [130, 7], [2047, 3],
         [3, 2047]]


@pytest.mark.parametrize("n", FFT + DENSE, ids=str)
def test_plane_sizes(A, n):  # noqa: F811
    cfg = cfg_of(3, n + [3])
    U = I.white_random(cfg, 71, amp=0.3)
    check(gpu_spectrum(A, cfg, U, 1), O.spectrum(cfg, U, 1))


@pytest.mark.parametrize("n", [1, 2, 8, 512, 2048, 3, 63, 129, 2047])
def test_line_sizes(A, n):  # noqa: F811
    cfg = cfg_of(2, [n, 5])
    U = I.white_random(cfg, 72, amp=0.3)
    check(gpu_spectrum(A, cfg, U, 3), O.spectrum(cfg, U, 3))
