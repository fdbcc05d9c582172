"""GPU: tables of five to eight materials, whose jobs run as passes, the electron pass of eight in workgroups of the ten
wavefronts that LDS has room for.  The tables hold four materials twice over, so that a phantom that picks either copy is
the same problem as one of four materials, which runs as a history pool: the same bits at every workgroup size."""
import numpy as np
import pytest

from paper_1101_1245_amd import gpumcd as G, inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("materials", [5, 7, 8])
@pytest.mark.parametrize("particle", [I.ELECTRON, I.PHOTON])
def test_materials_twice_over(materials, particle):
    ph = I.ellipsoids((21, 18, 25), 0.5, seed=9)
    src = I.centred(ph, I.Source(particle, e=10.0, wx=4.0, wy=3.0))
    phys = I.Physics(ecut=0.7, pcut=0.05)
    with G.Context(0) as c:
        pid, tid = c.load_phantom(ph), c.load_tables(I.DEFAULT_MATERIALS, phys)
        want = c.run_beam(pid, tid, src, 60_000, 3)
        assert want[2]["n_round_launches"] == 1
        copy = np.random.default_rng(1).random(ph.mat.shape) < 0.5
        twice = I.Phantom(ph.rho, np.where(copy & (ph.mat + 4 < materials), ph.mat + 4, ph.mat).astype(np.uint8), ph.voxel)
        pid = c.load_phantom(twice)
        tid = c.load_tables((I.DEFAULT_MATERIALS + I.DEFAULT_MATERIALS)[:materials], phys)
        for wg in (0, 64, 256, 640, 1024):
            d, s, st = c.run_beam(pid, tid, src, 60_000, 3, tuning={"wg_size": wg})
            assert st["n_electron_launches"] > 0 and st["n_round_launches"] == 0 and st["ledger_residual_lsb"] == 0
            assert np.array_equal(d, want[0]) and np.array_equal(s, want[1]), wg
            assert st["n_e_steps"] == want[2]["n_e_steps"]
