"""Response right-hand sides over several blocks of eight bands, with workgroups
that take units of more than one k-point and block.  Bound as in the module the
cases come from."""
import pytest

from test_gpu_rhs_units import test_rhs_shares as _shares

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nk,ecut,nocc", [(130, 9.0, 17), (90, 9.0, 24), (70, 12.0, 33), (2, 30.0, 64), (1, 35.0, 40)])
def test_bands(nk, ecut, nocc):
    _shares(nk, ecut, nocc)
