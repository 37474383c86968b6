"""Structure functions at the edges of their tiles: line lengths where the lines per
tile change, separations past a line's end, more separations than one launch takes."""
import numpy as np
import pytest

from oracle import stats as ST
from tests.helpers import forced_modes, gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("shape,rs", [
    ((1, 1, 1), [1]),
    ((5, 1, 3), [1, 2, 3]),
    ((6, 7, 257), [1, 200, 256, 257, 258]),
    ((3, 513, 9), list(range(1, 18))),
    ((1025, 4, 6), [1, 1024]),
    ((4, 6, 2048), [5, 2047, 4097]),
    ((3, 2049, 5), [1, 2, 2048]),
    ((2, 3, 2100), [7]),
    ((40, 48, 56), [1, 2, 3, 4, 6, 8, 11, 16, 23, 32, 40, 47, 48, 55, 56, 57, 2**31 - 1] * 2),
])
def test_structure_functions_match_oracle(shape, rs):
    """FP64, against the oracle on the same velocity.  The sums of up to n = 3 cells
    terms of like size differ by their order only: n 2^-53 of the sum of magnitudes at
    most, 1e-10 here; the odd signed moment cancels, so its bar is set by |du|^3."""
    from paper_2512_23116_amd import lbm
    lat = lbm.Lattice(shape, 0.52, 0.13, forced_modes(F0=3e-5, seed=4), precision="fp64",
                      smag_form=1)
    lat.init(lbm.LBM_INIT_NOISE, 0.03, 11)
    lat.step(2)
    _, u = lat.moments()
    S = lat.structure_functions(rs)
    lat.close()
    ref = ST.structure_functions(u, rs)
    scale = ref.copy()
    scale[:, 1] = ref[:, 2]
    np.testing.assert_array_less(np.abs(S - ref), 1e-10 * scale + 1e-300)
