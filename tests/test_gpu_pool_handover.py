"""GPU: jobs whose cascades overfill the history pool's stacks.  With the stacks cut to their least size an ordinary deep
cascade does it: the pool gives the job up (one launch, discarded) and it runs as passes, with the same bits, in the plain,
batched and served forms; the tallies, marks, counters and buffers it leaves serve the next job.  At their own size the
stacks hold the deepest cascades that the host's rule lets into the pool."""
import numpy as np
import pytest

from paper_1101_1245_amd import gpumcd as G, inputs as I

pytestmark = pytest.mark.gpu
PASSES = {"rounds_per_check": 5}      # any knob of the passes away from its default
LOW = I.Physics(ecut=0.05, pcut=0.01)                # some 25 delta rays per electron wait on a stack
COUNTS = ("n_e_steps", "n_photon_events", "n_photon_interactions", "n_fictitious", "n_hard", "n_secondaries", "e_in_mev",
          "e_dep_mev", "e_esc_mev", "e_sink_mev", "s_rel", "ledger_residual_lsb")


@pytest.fixture(scope="module")
def ctx():
    with G.Context(0) as c:
        yield c


@pytest.fixture()
def small():
    with G.Context(0) as c:
        c.pool_check(640)
        yield c


def load(c, ph, physics=LOW):
    return c.load_phantom(ph), c.load_tables((I.WATER,), physics)


def pooled(st):
    return st["n_round_launches"] == 1 and st["n_electron_launches"] == 0


def same(a, b):
    for x, y in zip(a[:-1], b[:-1]):
        assert np.array_equal(x, y) and x.max() > 0
    for k in COUNTS:
        assert a[-1][k] == b[-1][k], k


# dense tallies; few words touched (cleared by the finalize); and fewer still (marked)
@pytest.mark.parametrize("side", [20, 64, 160])
@pytest.mark.parametrize("out", ["numpy", "torch"])
def test_plain_job_is_handed_over(ctx, small, side, out):
    ph = I.homogeneous(side, 32.0 / side)
    src = I.centred(ph, I.Source(I.ELECTRON, e=20.0, wx=4.0, wy=4.0))
    n = 200_000
    a, b = load(small, ph), load(ctx, ph)
    for _ in range(2):
        before = small.pool_check()
        r = small.run_beam(*a, src, n, 9, out=out)
        assert small.pool_check() == before + 1 and not pooled(r[-1]) and r[-1]["n_electron_launches"] > 0
        r = [x.cpu().numpy() if hasattr(x, "cpu") else x for x in r]
        same(r, ctx.run_beam(*b, src, n, 9, tuning=PASSES))
        # a job that fits, on the workspace that the other left
        r = small.run_beam(*a, src, 500, 4)
        assert pooled(r[-1])
        same(r, ctx.run_beam(*b, src, 500, 4, tuning=PASSES))
    ta, _ = small.run_beam_tally(*a, src, n, 9)
    tb, _ = ctx.run_beam_tally(*b, src, n, 9, tuning=PASSES)
    assert np.array_equal(ta, tb)
    for h in b:
        ctx.release(h)


@pytest.mark.parametrize("side", [20, 160])
@pytest.mark.parametrize("sigma", [True, False])
@pytest.mark.parametrize("out", ["numpy", "torch"])
def test_batched_job_is_handed_over(ctx, small, side, sigma, out):
    ph = I.homogeneous(side, 32.0 / side)
    beams = [I.centred(ph, I.Source(p, e=20.0, wx=4.0, wy=4.0, beam_id=i)) for i, p in enumerate((I.ELECTRON, I.PHOTON))]
    n = [150_000, 20_000 if sigma else 20]      # 20 histories: no batches of its own for each beam
    a, b = load(small, ph), load(ctx, ph)
    before = small.pool_check()
    kw = dict(per_beam=True, per_beam_sigma=sigma)
    r = small.run_beams(*a, beams, n, 9, out=out, tuning={}, **kw)
    assert small.pool_check() == before + 1 and not pooled(r[-1])
    r = [x.cpu().numpy() if hasattr(x, "cpu") else x for x in r if x is not None]
    same(r, [x for x in ctx.run_beams(*b, beams, n, 9, tuning=PASSES, **kw) if x is not None])
    for h in b:
        ctx.release(h)


@pytest.mark.parametrize("side", [20, 160])
def test_served_request_is_handed_over(ctx, small, side):
    ph = I.homogeneous(side, 32.0 / side)
    src = I.centred(ph, I.Source(I.ELECTRON, e=20.0, wx=4.0, wy=4.0))
    a, b = load(small, ph), load(ctx, ph)
    small.server_start(max_slots=1)
    counts = (200_000, 500, 300_000, 500)       # the small ones fit
    got = [small.poll(t) for t in [small.submit(*a, src, n, 9) for n in counts]]
    small.server_stop()
    for n, (done, d, s, st) in zip(counts, got):
        assert done and pooled(st) == (n == 500)
        same((d, s, st), ctx.run_beam(*b, src, n, 9, tuning=PASSES))
    for h in b:
        ctx.release(h)


@pytest.mark.parametrize("particle", [I.ELECTRON, I.PHOTON])
def test_stacks_hold_what_the_rule_lets_in(ctx, particle):
    ph = I.homogeneous((20, 20, 30), 1.0)
    src = I.centred(ph, I.Source(particle, e=30.0, wx=1.0, wy=1.0))
    pid, tid = load(ctx, ph)                    # K_cut just above 0.0016 of the energy
    r = ctx.run_beam(pid, tid, src, 600_000, 9)
    assert pooled(r[-1])
    same(r, ctx.run_beam(pid, tid, src, 600_000, 9, tuning=PASSES))
    ctx.release(pid)
    ctx.release(tid)


def test_stack_sizes_are_checked(ctx):
    for n in (-64, 1, 576, 700, 4160):
        with pytest.raises(G.GpumcdError) as e:
            ctx.pool_check(n)
        assert e.value.code == G.GMC_EINVAL


def test_long_served_request_is_handed_over_after_one_launch(ctx, small):
    ph = I.homogeneous(20, 1.6)
    src = I.centred(ph, I.Source(I.ELECTRON, e=20.0, wx=4.0, wy=4.0))
    n = 3 * (1 << 22) + 77                      # four launches in the pool
    a, b = load(small, ph), load(ctx, ph)
    small.server_start(max_slots=1)
    before = small.pool_check()
    done, d, s, st = small.poll(small.submit(*a, src, n, 9))
    assert done and not pooled(st) and small.pool_check() == before + 1
    got = small.poll(small.submit(*a, src, 500, 9))
    small.server_stop()
    assert pooled(got[-1]) and small.pool_check() == before + 2
    same((d, s, st), ctx.run_beam(*b, src, n, 9, tuning=PASSES))
    same(got[1:], ctx.run_beam(*b, src, 500, 9, tuning=PASSES))
    for h in b:
        ctx.release(h)
