"""The collision's folded coefficients and explicit fused multiply-adds: every
relaxation rate against the oracle, and the same bits in every kernel that
collides."""
import ctypes

import numpy as np
import pytest

from oracle import init_fields as I
from tests.helpers import W4, forced_modes, gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

RATES = [dict(s_e=1.19, s_eps=1.4, s_q=1.2, s_pi=1.4, s_m=1.98),
         dict(s_e=0.7, s_eps=1.9, s_q=1.7, s_pi=0.9, s_m=1.1),
         dict(s_e=1.0, s_eps=1.0, s_q=1.0, s_pi=1.0, s_m=1.0)]


@pytest.fixture(scope="module")
def lbm():
    from paper_2512_23116_amd import lbm as m
    m.lib()
    return m


@pytest.mark.parametrize("rates", RATES)
@pytest.mark.parametrize("streaming,tau_mode,rho0", [("aa", 0, 1.0), ("ab", 1, 1.0), ("ab", 0, 1.3)])
def test_every_relaxation_rate_against_the_oracle(lbm, orc, rates, streaming, tau_mode, rho0):
    """FP64, two steps (AA even and odd) on a ragged lattice; the one-step bar of
    1e-12 holds for both with room (each step rounds at 1e-16 of the populations)."""
    nz, ny, nx = shape = (7, 9, 11)
    modes = forced_modes(F0=3e-4, seed=2)
    cfg = lbm.lbm_config_default()
    cfg.nx, cfg.ny, cfg.nz = nx, ny, nz
    cfg.precision, cfg.streaming = lbm.LBM_FP64, lbm.STREAMING[streaming]
    cfg.tau0, cfg.smag_C, cfg.rho0, cfg.tau_mode = 0.507, 0.13, rho0, tau_mode
    for name, v in rates.items():
        setattr(cfg, name, v)
    table = lbm.make_modes(modes)
    cfg.n_force_modes = len(modes)
    cfg.force_modes = ctypes.cast(table, ctypes.POINTER(lbm.lbm_force_mode))
    h = lbm.lbm_create(cfg)
    olat = orc.Lattice(shape, 0.507, 0.13, modes, rho0=rho0, tau_mode=tau_mode, **rates)
    ref = olat.init(I.KIND_NOISE, 0.05, 3)
    lbm.lbm_set_populations(h, ref.reshape(19, -1))
    lbm.lbm_step(h, 2)
    got = lbm.lbm_get_populations(h, nx * ny * nz).reshape(ref.shape)
    lbm.lbm_destroy(h)
    ref = olat.step(ref, 2)
    scale = np.abs(ref.reshape(19, -1) - rho0 * W4.reshape(19, 1)).max()
    assert np.abs(got - ref).max() <= 1e-12 * scale


@pytest.mark.parametrize("precision", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("shape", [(5, 17, 62), (9, 15, 63), (4, 14, 125),
                                   (5, 13, 64), (4, 14, 128), (3, 27, 32), (6, 15, 192),
                                   (4, 14, 31), (5, 15, 93)])
def test_two_steps_per_pass_give_the_bits_of_single_steps(lbm, precision, shape):
    """Lattices of one tile, one column or row more, and several tiles, of rows in whole
    cache lines and not (the two tile shapes): the two-step
    kernel, single A/B steps and AA steps agree bit for bit."""
    out = []
    for streaming, tb in (("ab", 2), ("ab", 0), ("aa", 0)):
        lat = lbm.Lattice(shape, 0.507, 0.12, forced_modes(F0=3e-5, seed=5), precision=precision,
                          streaming=streaming, smag_form=1, temporal_block=tb, steps_per_graph=0)
        lat.init(lbm.LBM_INIT_NOISE, 0.03, 6)
        lat.step(6)
        out.append(lat.populations())
        lat.close()
    np.testing.assert_array_equal(out[0], out[1])
    np.testing.assert_array_equal(out[1], out[2])
