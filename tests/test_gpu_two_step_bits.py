"""Two steps per pass give the bits of single steps on deep lattices too: several
chunks of planes and both tile shapes, through a captured graph and plain launches,
with every collision option."""
import numpy as np
import pytest

from tests.helpers import forced_modes, gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _states(shape, precision, modes, C, smag_form, tau_mode, spg, steps, read):
    from paper_2512_23116_amd import lbm
    out = []
    for tb in (0, 2):
        lat = lbm.Lattice(shape, 0.507, C, modes, precision=precision, streaming="ab",
                          smag_form=smag_form, tau_mode=tau_mode, temporal_block=tb,
                          steps_per_graph=spg)
        lat.init(lbm.LBM_INIT_NOISE, 0.03, 7)
        for n in steps:
            lat.step(n)
        out.append(read(lat))
        lat.close()
    return out


@pytest.mark.parametrize("spg", [0, 8])
@pytest.mark.parametrize("precision", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("shape", [(67, 29, 64), (70, 27, 93), (131, 15, 40), (64, 64, 128)])
def test_deep_lattices(shape, precision, spg):
    modes = forced_modes(F0=3e-5, seed=8)
    a, b = _states(shape, precision, modes, 0.12, 1, 0, spg, (2, 1, 3, 24, 19),
                   lambda lat: lat.populations())
    np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("C,smag_form,tau_mode,forced", [(0.0, 1, 0, True), (0.12, 0, 0, True),
                                                         (0.12, 1, 1, True), (0.3, 0, 1, False)])
@pytest.mark.parametrize("precision", ["fp32", "fp16", "bf16"])
def test_every_collision_option(C, smag_form, tau_mode, forced, precision):
    modes = forced_modes(F0=3e-5, seed=13) if forced else ()
    for nx in (64, 70):
        a, b = _states((37, 31, nx), precision, modes, C, smag_form, tau_mode, 8, (2, 1, 3, 24),
                       lambda lat: lat.populations())
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("precision", ["fp32", "fp16"])
def test_large_lattice(precision):
    cells = np.random.default_rng(0).integers(0, 256 ** 3, 20000)
    a, b = _states((256, 256, 256), precision, forced_modes(F0=1e-5, seed=3), 0.1, 1, 0, 64,
                   (66,), lambda lat: lat.sample(cells))
    np.testing.assert_array_equal(a, b)
