"""GPU: the round kernel's grid -- as many wavefronts on a CU whatever the workgroup, the default workgroup the largest --
at the edges of the workgroup sizes and at loads below and above a chunk per wavefront: the passes' bits."""
import numpy as np
import pytest

from paper_1101_1245_amd import gpumcd as G, inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    with G.Context(0) as c:
        yield c


@pytest.mark.parametrize("materials", [1, 4])
@pytest.mark.parametrize("n", [64, 40_000, 300_000])
def test_round_kernel_at_every_workgroup_size(ctx, materials, n):
    ph = I.ellipsoids((21, 18, 25), 0.5, seed=9) if materials == 4 else I.homogeneous((21, 18, 25), 0.5)
    tid, pid = ctx.load_tables(I.DEFAULT_MATERIALS[:materials], I.Physics(ecut=0.7, pcut=0.05)), ctx.load_phantom(ph)
    for particle in (I.ELECTRON, I.PHOTON):
        src = I.centred(ph, I.Source(particle, e=6.0, wx=4.0, wy=3.0))
        want = ctx.run_beam(pid, tid, src, n, 3, tuning={"rounds_per_check": 5})
        for wg in (0, 64, 128, 448, 512, 1024):
            d, s, st = ctx.run_beam(pid, tid, src, n, 3, tuning={"persistent": 1, "wg_size": wg})
            assert st["n_round_launches"] > 0 and st["n_electron_launches"] == 0
            assert np.array_equal(d, want[0]) and np.array_equal(s, want[1]), wg
            assert st["n_e_steps"] == want[2]["n_e_steps"] and st["ledger_residual_lsb"] == 0
    ctx.release(pid)
    ctx.release(tid)
