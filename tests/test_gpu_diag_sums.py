"""Every sum of the diagnostics where waves and blocks are partly filled."""
import numpy as np
import pytest

from tests.helpers import forced_modes, gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 1, 63), (5, 13, 1), (3, 5, 17), (1, 257, 1),
                                   (7, 11, 13)])
def test_statistics_of_few_cells(shape):
    """1, 63, 65, 255, 257 and 1001 cells, FP64: the sums of the library's own velocity
    and density, and of the oracle's strain and theta of the same state.  The terms
    agree to 1e-13 and the sums' order moves them by n 2^-53; bars 1e-11 of the sums of
    magnitudes (|S|^2 comes from differences of populations)."""
    from oracle import ref_numpy as R
    from paper_2512_23116_amd import lbm
    modes = forced_modes(F0=4e-5, seed=5)
    lat = lbm.Lattice(shape, 0.507, 0.15, modes, precision="fp64", smag_form=1)
    lat.init(lbm.LBM_INIT_NOISE, 0.03, 13)
    lat.step(2)
    st, f = lat.stats(), lat.populations()
    rho, u = lat.moments()
    lat.close()
    F = R.force_field(shape, modes)
    _, info = R.collide(f, F, 0.507, 0.15, smag_form=1)
    theta = info["tau_e"] - 0.5

    def near(got, terms):
        assert abs(got - terms.mean()) <= 1e-11 * np.abs(terms).mean() + 1e-18, (got, terms.mean())

    assert st["n_nonfinite"] == 0 and st["n_cells"] == rho.size
    near(st["mass"] / rho.size, rho)
    near(st["energy"], 0.5 * (u * u).sum(0))
    near(st["energy_rho"], 0.5 * rho * (u * u).sum(0))
    near(st["injection"], (F * u).sum(0))
    for a in range(3):
        near(st["momentum"][a] / rho.size, rho * u[a])
        near(st["u_mean"][a], u[a])
    for k, (a, b) in enumerate(((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))):
        near(st["uu"][k], u[a] * u[b])
    near(st["theta_mean"], theta)
    assert abs(st["theta_min"] - theta.min()) <= 1e-11 * theta.min()
    assert abs(st["theta_max"] - theta.max()) <= 1e-11 * theta.max()
