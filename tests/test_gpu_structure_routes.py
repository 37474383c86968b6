"""Structure functions on both sides of the rule that sends few separations past LDS:
tiny lattices, short rows, up to 4 separations of 5e6 cells in all."""
import numpy as np
import pytest

from oracle import stats as ST
from tests.helpers import forced_modes, gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("shape,counts", [((34, 34, 34), (2, 16, 17)), ((34, 34, 35), (2, 4, 5)),
                                          ((80, 80, 7), (8, 9)), ((80, 80, 15), (5, 6)),
                                          ((60, 60, 16), (4, 5)), ((136, 136, 136), (2, 3)),
                                          ((137, 135, 137), (3,))])
def test_few_separations(shape, counts):
    """FP64 against the oracle on the same velocity, bars as for the tiles: n 2^-53 of the
    sum of magnitudes at most for sums of n = 3 cells terms, 1e-10 here."""
    from paper_2512_23116_amd import lbm
    lat = lbm.Lattice(shape, 0.52, 0.13, forced_modes(F0=3e-5, seed=4), precision="fp64",
                      smag_form=1)
    lat.init(lbm.LBM_INIT_NOISE, 0.03, 14)
    lat.step(2)
    _, u = lat.moments()
    rs = [1, 2, 3, 5, 7, 9, 12, 15, 18, 20, 24, 30, 33, 34, 35, 40, 80][:max(counts)]
    ref = ST.structure_functions(u, rs)
    scale = ref.copy()
    scale[:, 1] = ref[:, 2]
    for n in counts:
        S = lat.structure_functions(rs[:n])
        np.testing.assert_array_less(np.abs(S - ref[:n]), 1e-10 * scale[:n] + 1e-300)
    lat.close()
