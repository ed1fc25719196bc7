"""The forward pass against the FP64 oracle on both sides of the lines between
the pixel sums and the node sums of the continuum moments, at last lanes of one
pixel and of all seventeen."""

import pytest

from test_gpu_moments import test_forward_matches_the_oracle_beside_each_line as check_forward

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]


@pytest.mark.parametrize("n_pix,degree", [
    (241, 4), (242, 4), (255, 4), (655, 6), (656, 6), (664, 6), (1228, 8), (1229, 8), (1242, 8),
    (1964, 10), (1965, 10), (1972, 10), (1973, 10), (1990, 10)])
def test_forward_beside_each_line(n_pix, degree):
    check_forward(n_pix, 64, degree)
