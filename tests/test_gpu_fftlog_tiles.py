"""FFTLog at the edges of its product kernel's tiles: one, two or four column tiles of angles with a
remainder, row tiles of coefficients with a remainder, k ranges shorter than the requests ahead,
one model and several; tolerance of the FFTLog parity tests."""

import pytest

from tests import test_gpu_fftlog as F

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ntheta", [2, 15, 16, 17, 32, 33, 48, 64, 65, 130])
@pytest.mark.parametrize("N,nchi,nmodels", [(4, 2, 1), (6, 31, 3), (30, 33, 2), (32, 64, 5), (62, 100, 1)])
def test_tile_edges(ntheta, N, nchi, nmodels):
    F._check("tile edges", N, 30.0, F.NU_DEFAULT, nchi, ntheta, nmodels, seed=7 * N + ntheta)
