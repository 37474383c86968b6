"""The theta histogram where its blocks and their shares of the cells begin and end."""
import numpy as np
import pytest

from tests.helpers import forced_modes, gpu_available
from tests.test_gpu_analysis import _bin_counts

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("shape", [(1, 1, 1), (11, 3, 31), (8, 8, 16), (5, 5, 41),
                                   (64, 64, 64), (5, 13, 4033)])
@pytest.mark.parametrize("nbins", [1, 4096])
def test_counts_at_block_edges(shape, nbins):
    """1, 1023, 1024, 1025, 2^18 and 2^18 + 1 cells, FP64: the counts of the oracle's
    theta of the same state, but for cells within 1e-13 of an edge (its rounding)."""
    from oracle import ref_numpy as R
    from paper_2512_23116_amd import lbm
    modes = forced_modes(F0=4e-5, seed=5)
    lat = lbm.Lattice(shape, 0.507, 0.15, modes, precision="fp64", smag_form=1)
    lat.init(lbm.LBM_INIT_NOISE, 0.03, 13)
    lat.step(1)
    _, info = R.collide(lat.populations(), R.force_field(shape, modes), 0.507, 0.15, smag_form=1)
    theta = (info["tau_e"] - 0.5).ravel()
    lo, hi = np.quantile(theta, 0.1), np.quantile(theta, 0.9) + 1e-6
    got = lat.theta_histogram(lo, hi, nbins)
    lat.close()
    q = (theta - lo) * (nbins / (hi - lo))
    near = (np.abs(q - np.round(q)) * (hi - lo) / nbins <= 1e-13 * np.abs(theta).max()).sum()
    assert got.sum() == theta.size
    assert np.abs(got - _bin_counts(theta, lo, hi, nbins)).sum() <= 2 * near
