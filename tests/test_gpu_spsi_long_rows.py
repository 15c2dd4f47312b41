"""S|psi> on rows of more than 1024 plane waves against the oracle's dense S, on
both sides of the 8 projectors that the smaller kernel holds.  Bounds as for S|psi>
elsewhere."""
import pytest

from test_gpu_spsi_tiles import test_tile_edges as _edges

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nbnd,nproj", [(6, 8), (2, 9)])
def test_long_rows(nbnd, nproj):
    _edges(70.0, nbnd, nproj)
