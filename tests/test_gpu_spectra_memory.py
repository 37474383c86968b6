"""What lbm_spectra_1d keeps on the handle."""
import numpy as np
import pytest
import torch

from tests.helpers import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("shape", [(16, 16, 16), (20, 24, 30)])
def test_many_bins(shape):
    """kmax 2048 on a small lattice: one component's partial sums (1024 blocks of 3 x 2049
    doubles, 50.4 MB); 8 MB are allowed beside them for the results and for what the
    allocations are rounded up to.  The bins of a shorter call are the same sums, of at
    most 1e4 modes each in another order: 1e4 x 2^-53."""
    from paper_2512_23116_amd import lbm
    lat = lbm.Lattice(shape, 0.51, 0.1, (), precision="fp32", streaming="aa")
    lat.init(lbm.LBM_INIT_NOISE, 0.02, 3)
    lat.step(2)
    few, _ = lat.spectra_1d(20, with_ic=False)
    free = torch.cuda.mem_get_info()[0]
    many, _ = lat.spectra_1d(2048, with_ic=False)
    kept = free - torch.cuda.mem_get_info()[0]
    lat.close()
    assert kept <= 1024 * 3 * 2049 * 8 + (8 << 20)
    np.testing.assert_allclose(many[:, :, :21], few, rtol=2e-12, atol=0)
    assert (many[:, :, 21:] == 0).all()
