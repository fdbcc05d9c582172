"""GPU: per-beam doses and uncertainties with more batches than the finalize's register forms hold, at the edges of the
batches it has in flight: device results (all beams in one launch) equal the host ones (a beam at a time), and a beam run
alone, bit for bit; twice in a row, for tallies that the finalize leaves at zero and tallies that it does not."""
import numpy as np
import pytest

from paper_1101_1245_amd import gpumcd as G, inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    with G.Context(0) as c:
        yield c


@pytest.mark.parametrize("K", [33, 35, 36, 100])
@pytest.mark.parametrize("n", [400, 40_000])            # few words touched, and most of them
@pytest.mark.parametrize("beams", [2, 9])
def test_beams_of_many_batches(ctx, K, n, beams):
    ph = I.homogeneous((13, 10, 11), 0.7)
    pid, tid = ctx.load_phantom(ph), ctx.load_tables((I.WATER,), I.Physics(ecut=0.7, pcut=0.05, n_batches=K))
    src = [I.centred(ph, I.Source(b % 2, e=4.0 + b, wx=2.0, wy=2.0, beam_id=b)) for b in range(beams)]
    counts = [n + 7 * b for b in range(beams)]
    for sigma in (True, False):
        kw = dict(tuning={}, per_beam=True, per_beam_sigma=sigma, sigma=sigma)
        host = ctx.run_beams(pid, tid, src, counts, 3, **kw)
        for _ in range(2):
            dev = ctx.run_beams(pid, tid, src, counts, 3, out="torch", **kw)
            for a, b in zip(host[:4], dev[:4]):
                assert (a is None and b is None) or np.array_equal(a, b.cpu().numpy())
        for b in range(beams):
            d, s, _ = ctx.run_beam(pid, tid, src[b], counts[b], 3, sigma=sigma)
            assert np.array_equal(host[0][b], d) and d.max() > 0
            assert not sigma or np.array_equal(host[1][b], s)
    ctx.release(pid)
    ctx.release(tid)
