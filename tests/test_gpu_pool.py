"""GPU: the history pool (one launch per job, wavefront-private stacks) against the pass engine, which an explicit knob
of the passes selects: doses, uncertainties, raw tallies and event counts are the same bits at the sizes where the pool's
claims, stacks and launches change -- a single batch of histories, one history per wavefront, a few, more than one claim
each, primaries that miss the phantom or start below the cutoff, several beams of both types, and cascades that overfill
a wavefront's stacks, which run as passes."""
import numpy as np
import pytest

from paper_1101_1245_amd import inputs as I

pytestmark = pytest.mark.gpu
PASSES = {"rounds_per_check": 5}      # any knob of the passes away from its default
COUNTS = ("n_e_steps", "n_photon_events", "n_photon_interactions", "n_fictitious", "n_hard", "n_secondaries", "e_in_mev",
          "e_dep_mev", "e_esc_mev", "e_sink_mev", "s_rel")


@pytest.fixture(scope="module")
def G():
    from paper_1101_1245_amd import gpumcd
    return gpumcd


@pytest.fixture(scope="module")
def ctx(G):
    c = G.Context(0)
    yield c
    c.close()


def pooled(st):
    return st["n_round_launches"] >= 1 and st["n_electron_launches"] == 0 and st["n_photon_launches"] == 0


def check(a, b, arrays):
    for i in range(arrays):
        assert (a[i] is None and b[i] is None) or np.array_equal(a[i], b[i]), i
    for k in COUNTS:
        assert a[-1][k] == b[-1][k] or (a[-1][k] != a[-1][k] and b[-1][k] != b[-1][k]), k
    assert pooled(a[-1]) and not pooled(b[-1]) and a[-1]["ledger_residual_lsb"] == 0


def run_both(ctx, mats, ph, src, physics, n, seed=3):
    tid, pid = ctx.load_tables(mats, physics), ctx.load_phantom(ph)
    try:
        a = ctx.run_beam(pid, tid, src, n, seed)
        check(a, ctx.run_beam(pid, tid, src, n, seed, tuning=PASSES), 2)
        ta, sta = ctx.run_beam_tally(pid, tid, src, n, seed)
        tb, _ = ctx.run_beam_tally(pid, tid, src, n, seed, tuning=PASSES)
        assert pooled(sta) and np.array_equal(ta, tb)
    finally:
        ctx.release(pid)
        ctx.release(tid)


@pytest.mark.parametrize("particle", [I.ELECTRON, I.PHOTON])
@pytest.mark.parametrize("n", [32, 63, 65, 2000, 4096 * 64 + 1, 4096 * 300 + 17])
def test_pool_history_counts(ctx, particle, n):
    ph = I.ellipsoids((33, 29, 41), 0.4, seed=5)
    src = I.centred(ph, I.Source(particle, I.TRIANGULAR, 10.0, e_lo=0.3, e_mode=10.0, e_hi=18.0, wx=5.0, wy=4.0,
                                 first_history=11))
    run_both(ctx, I.DEFAULT_MATERIALS, ph, src, I.Physics(ecut=0.7, pcut=0.01), n)


@pytest.mark.parametrize("kw", [
    {"wx": 40.0, "wy": 40.0},                       # most primaries miss the phantom
    {"e": 0.3, "wx": 3.0, "wy": 3.0},               # electrons below the cutoff deposit where they enter
    {"e": 29.5, "wx": 0.1, "wy": 0.1},
], ids=["wide", "sub-cutoff", "30MeV-pencil"])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_pool_primaries_and_modes(ctx, kw, mode):
    ph = I.homogeneous((16, 16, 24), 0.5)
    for particle in (I.ELECTRON, I.PHOTON):
        src = I.centred(ph, I.Source(particle, **{"e": 6.0, **kw}))
        run_both(ctx, (I.WATER,), ph, src, I.Physics(ecut=0.7, pcut=0.01, test_mode=mode, esmax_gcm2=0.11 * mode), 30_000)


@pytest.mark.parametrize("per_beam,sigma", [(False, False), (True, False), (True, True)])
@pytest.mark.parametrize("beams", [2, 300])          # the beam table in LDS, and beyond it
def test_pool_several_beams(ctx, beams, per_beam, sigma):
    j = I.beamlet_job(n_beamlets=beams, shape=(40, 40, 32), voxel=0.5, count_scale=0.01, min_count=64)
    tid, pid = ctx.load_tables(j.materials, j.physics), ctx.load_phantom(j.phantom)
    try:
        kw = dict(per_beam=per_beam, per_beam_sigma=sigma)
        a = ctx.run_beams(pid, tid, j.sources, j.counts, 2, tuning={}, **kw)
        check(a, ctx.run_beams(pid, tid, j.sources, j.counts, 2, tuning=PASSES, **kw), 4)
    finally:
        ctx.release(pid)
        ctx.release(tid)


def test_deep_cascades_run_as_passes(ctx):
    # K_cut below 0.0016 of the beam energy: by rule; just above it with a thick, low-cutoff phantom: the pool, which
    # hands the job over if its stacks could overflow
    ph = I.homogeneous((20, 20, 30), 1.0)
    for ecut, n in ((0.01, 200), (0.05, 20_000)):
        src = I.centred(ph, I.Source(I.ELECTRON, e=30.0, wx=1.0, wy=1.0))
        tid, pid = ctx.load_tables((I.WATER,), I.Physics(ecut=ecut, pcut=0.001)), ctx.load_phantom(ph)
        try:
            a = ctx.run_beam(pid, tid, src, n, 9)
            b = ctx.run_beam(pid, tid, src, n, 9, tuning=PASSES)
            assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
            assert a[2]["n_secondaries"] == b[2]["n_secondaries"] and a[2]["ledger_residual_lsb"] == 0
            if ecut == 0.01:
                assert not pooled(a[2])
        finally:
            ctx.release(pid)
            ctx.release(tid)


def test_served_requests_of_several_pool_launches(ctx, G):
    ph = I.homogeneous(24, 0.5)
    n = (1 << 22) + 12_345          # a second launch with a remainder
    src = I.centred(ph, I.Source(I.PHOTON, e=2.0, wx=3.0, wy=3.0))
    tid, pid = ctx.load_tables((I.WATER,), I.Physics(ecut=0.7, pcut=0.01)), ctx.load_phantom(ph)
    with G.Context(0) as c2:
        t2, p2 = c2.load_tables((I.WATER,), I.Physics(ecut=0.7, pcut=0.01)), c2.load_phantom(ph)
        c2.server_start(max_slots=2)
        tickets = [c2.submit(p2, t2, src, m, 4) for m in (n, 5000, n)]
        got = [c2.poll(t) for t in tickets]
        c2.server_stop()
    try:
        for (_, d, s, st), m in zip(got, (n, 5000, n)):
            ref = ctx.run_beam(pid, tid, src, m, 4, tuning=PASSES)
            assert np.array_equal(d, ref[0]) and np.array_equal(s, ref[1])
            assert st["n_round_launches"] == -(-m // (1 << 22)) and st["ledger_residual_lsb"] == 0
    finally:
        ctx.release(pid)
        ctx.release(tid)


# around the histories at which the grid changes: a wavefront each up to four per CU (256 CUs), 64 each after that, in
# workgroups of 4, 8 and 16 wavefronts, until the grid is full
@pytest.mark.parametrize("n", [1021, 1025, 64 * 1024 - 1, 64 * 1024 + 65, 64 * 2048 + 63, 64 * 2048 + 64, 64 * 4096 + 129])
def test_pool_grid_edges(ctx, n):
    ph = I.ellipsoids((21, 18, 25), 0.5, seed=9)
    src = I.centred(ph, I.Source(I.ELECTRON, I.MONO, 6.0, wx=4.0, wy=3.0))
    run_both(ctx, I.DEFAULT_MATERIALS, ph, src, I.Physics(ecut=0.7, pcut=0.05), n)
