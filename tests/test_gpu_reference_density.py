"""A lattice of reference density 2^p with populations and force times 2^p steps
like that of density 1, scaled: factors of two do not round."""
import ctypes

import numpy as np
import pytest

from oracle import init_fields as I
from tests.helpers import W4, forced_modes, gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

SHAPE = (6, 9, 70)


def _steps(lbm, f, p, precision, scale, streaming, tb, tau_mode, n):
    nz, ny, nx = SHAPE
    modes = [(k, tuple(2.0 ** p * x for x in amp), phase)
             for k, amp, phase in forced_modes(F0=3e-4, seed=2)]
    cfg = lbm.lbm_config_default()
    cfg.nx, cfg.ny, cfg.nz = nx, ny, nz
    cfg.precision, cfg.streaming = lbm.PRECISION[precision], lbm.STREAMING[streaming]
    cfg.tau0, cfg.smag_C, cfg.rho0, cfg.tau_mode = 0.507, 0.2, 2.0 ** p, tau_mode
    cfg.temporal_block, cfg.storage_scale, cfg.steps_per_graph = tb, scale, 0
    table = lbm.make_modes(modes)
    cfg.n_force_modes = len(modes)
    cfg.force_modes = ctypes.cast(table, ctypes.POINTER(lbm.lbm_force_mode))
    h = lbm.lbm_create(cfg)
    lbm.lbm_set_populations(h, f.reshape(19, -1) * 2.0 ** p)
    lbm.lbm_step(h, n)
    out = lbm.lbm_get_populations(h, nx * ny * nz) * 2.0 ** -p
    lbm.lbm_destroy(h)
    return out


@pytest.mark.parametrize("tau_mode", [0, 1])
@pytest.mark.parametrize("precision,scale,streaming,tb,p", [
    ("fp32", 0.0, "aa", 0, 70), ("fp32", 0.0, "ab", 0, -70), ("fp32", 0.0, "ab", 2, 70),
    ("fp32", 0.0, "ab", 2, -70), ("bf16", 1024.0, "aa", 0, 60), ("bf16", 1024.0, "ab", 2, -70)])
def test_steps_do_not_depend_on_the_unit_of_density(orc, precision, scale, streaming, tb, p, tau_mode):
    """Each step forms the same products times a power of two.  The strain norm alone is
    rounded in other places there: three roundings of tau_e - tau0 more, which moves a
    population by less than its own rounding does.  So 4 steps differ by at most two
    roundings of the stored population a step."""
    from paper_2512_23116_amd import lbm
    olat = orc.Lattice(SHAPE, 0.507, 0.2, [], tau_mode=tau_mode)
    f = olat.init(I.KIND_NOISE, 0.05, 3)
    a = _steps(lbm, f, 0, precision, scale, streaming, tb, tau_mode, 4)
    b = _steps(lbm, f, p, precision, scale, streaming, tb, tau_mode, 4)
    unit = {"fp32": 2.0 ** -24, "bf16": 2.0 ** -8}[precision]
    assert np.isfinite(b).all()
    assert np.abs(a - b).max() <= 8 * unit * np.abs(a - W4.reshape(19, 1)).max()
