"""GPU parity of the compile-time transform lengths that are not multiples of
12: odd and twice-odd lines in theta and in z, most of whose stages have no
affine addresses.  Same checks and bars as for the multiples of 12."""
import pytest

import test_gpu_lengths as lengths

pytestmark = pytest.mark.gpu

# (N_r, M_theta, K + 1): theta lengths 3 M_theta, z lengths 3 (K + 1)
GRIDS = [(9, 5, 150), (9, 6, 135), (10, 9, 125), (9, 10, 90), (9, 15, 81), (11, 18, 75), (9, 25, 54), (9, 27, 50),
         (9, 30, 45), (10, 45, 30), (9, 50, 27), (9, 54, 25), (9, 75, 18), (9, 81, 15), (9, 90, 10), (9, 125, 9),
         (9, 135, 6), (9, 150, 5)]


@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("Ra", [0.0, 1.0e4])
def test_nonlinear_odd_lengths(grid, Ra):
    lengths.test_nonlinear_lengths(grid, Ra)


@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("Ra", [0.0, 1.0e4])
def test_nonlinear_vjp_odd_lengths(grid, Ra):
    lengths.test_nonlinear_vjp_lengths(grid, Ra)
