"""One-dimensional spectra on both sides of the size up to which the three transforms
go in one call."""
import numpy as np
import pytest

from oracle import stats as ST
from tests.helpers import forced_modes, gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("shape", [(64, 512, 511), (64, 512, 512)])
def test_spectra_1d_at_the_batch_limit(shape):
    """2^24 - 2^15 and 2^24 cells against the oracle on the same velocity; the bars of
    the small lattices' test (rounding of the transform, log2 n times 2^-53)."""
    from paper_2512_23116_amd import lbm
    lat = lbm.Lattice(shape, 0.52, 0.13, forced_modes(F0=3e-5, seed=4), precision="fp32",
                      smag_form=1)
    lat.init(lbm.LBM_INIT_NOISE, 0.02, 23)
    _, u = lat.moments()
    E, _ = lat.spectra_1d(9, with_ic=False)
    again, _ = lat.spectra_1d(9, with_ic=False)
    lat.close()
    ref = ST.one_dimensional_spectra(u)[:, :, :10]
    np.testing.assert_array_equal(E, again)
    np.testing.assert_allclose(E, ref, rtol=1e-10, atol=1e-14 * ref.max())
