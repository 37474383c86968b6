"""The theta histogram of small lattices, in blocks of 256 cells."""
import pytest

from tests.helpers import gpu_available
from tests.test_gpu_theta_hist import test_counts_at_block_edges as counts

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("shape", [(5, 3, 17), (4, 8, 8), (1, 1, 257), (40, 40, 25), (13, 17, 181)])
def test_counts(shape):
    """255, 256, 257, 40000 and 40001 cells, on both sides of the larger blocks."""
    counts(shape, 300)
