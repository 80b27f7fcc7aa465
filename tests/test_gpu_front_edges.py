"""Front kernels where their rules change, against dense references: large
fronts with fewer columns than a block of 16."""
import numpy as np
import pytest

from paper_2606_04725_amd import nmpc as N
from test_gpu_fronts import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G,H", [(24, 4), (16, 14)])
def test_narrow_large_front(G, H):
    """A panel of fewer than 16 columns at the top of a large front."""
    m, w = _check(N.Problem(N.plate_structure(G, H, 0.01)), 3 * G + H, f"plate {G} x {G} x {H}")
    assert np.any((m > 200) & (w < 16))
