"""Structure functions of lines of 512 cells (tiles of 16 lines), asked for alone and
in lists of any length."""
import numpy as np
import pytest

from oracle import stats as ST
from tests.helpers import forced_modes, gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("shape", [(6, 40, 512), (5, 512, 37), (512, 20, 18)])
def test_lists_of_separations(shape):
    """The same list gives the same bits, and a separation the same sums whatever list it
    is in, but for their order: n = 3 cells terms, n 2^-53 of the sum of magnitudes at
    most (1e-10; the odd signed moment cancels, its bar is set by |du|^3)."""
    from paper_2512_23116_amd import lbm
    lat = lbm.Lattice(shape, 0.52, 0.13, forced_modes(F0=3e-5, seed=4), precision="fp64",
                      smag_form=1)
    lat.init(lbm.LBM_INIT_NOISE, 0.03, 12)
    lat.step(2)
    _, u = lat.moments()
    rs = [1, 2, 3, 5, 8, 13, 21, 34, 55, 89, 144, 200, 255, 256, 300, 511, 512]
    ref = ST.structure_functions(u, rs)
    scale = ref.copy()
    scale[:, 1] = ref[:, 2]
    for n in (1, 2, 3, 5, 8, 9, 13, 16, 17):
        S = lat.structure_functions(rs[:n])
        np.testing.assert_array_equal(lat.structure_functions(rs[:n]), S)
        np.testing.assert_array_less(np.abs(S - ref[:n]), 1e-10 * scale[:n] + 1e-300)
    lat.close()
