"""GPU: a context's tallies are reused from job to job, cleared by the finalize that read them or by the next job.  A job
gives the same bits after any other -- sparse and dense ones, larger and smaller grids, jobs with per-beam results to
device and host memory, with some beams' results not asked for, more batches than the register finalize holds, raw
tallies, and a job that failed -- as in a new context."""
import numpy as np
import pytest

from paper_1101_1245_amd import inputs as I

pytestmark = pytest.mark.gpu


def jobs():
    """name -> function of a context that runs it and returns arrays to compare."""
    big, small = I.ellipsoids((70, 61, 50), 0.4, seed=2), I.ellipsoids((19, 22, 17), 0.5, seed=3)

    def one(ph, n, K=32, tally=False):
        def f(ctx):
            tid = ctx.load_tables(I.DEFAULT_MATERIALS, I.Physics(ecut=0.7, pcut=0.01, n_batches=K))
            pid = ctx.load_phantom(ph)
            src = I.centred(ph, I.Source(I.PHOTON, e=8.0, wx=4.0, wy=4.0))
            r = ctx.run_beam_tally(pid, tid, src, n, 5) if tally else ctx.run_beam(pid, tid, src, n, 5)
            ctx.release(pid)
            ctx.release(tid)
            return [x for x in r[:-1] if x is not None]
        return f

    def beams(ph, nb, n, K, per_beam, sigma, out, some=False):
        def f(ctx):
            from paper_1101_1245_amd import gpumcd as G
            import ctypes as C
            tid = ctx.load_tables(I.DEFAULT_MATERIALS, I.Physics(ecut=0.7, pcut=0.01, n_batches=K))
            pid = ctx.load_phantom(ph)
            srcs = [I.centred(ph, I.Source(b % 2, e=5.0 + b % 15, wx=0.5, wy=0.5, beam_id=b)) for b in range(nb)]
            if some:   # every other beam's dose only, through the C entry point
                keep, n_vox = [], ph.rho.size
                s = (G.gmc_source * nb)(*[G._src(x, keep) for x in srcs])
                d, pb = np.zeros(n_vox), np.zeros((nb, n_vox))
                rows = (C.c_void_p * nb)(*[pb[b].ctypes.data if b % 2 else None for b in range(nb)])
                st, tu = G.gmc_run_stats(), G.gmc_tuning()
                ctx._check(ctx._L.gmc_run_beams(ctx._h, pid, tid, s, (C.c_uint64 * nb)(*[n] * nb), nb, 5, rows, None,
                                                d.ctypes.data, None, G.GMC_HOST, C.byref(tu), C.byref(st)))
                r = [d, pb]
            else:
                r = ctx.run_beams(pid, tid, srcs, [n] * nb, 5, tuning={}, per_beam=per_beam, per_beam_sigma=sigma, out=out)
                r = [x if out == "numpy" else x.cpu().numpy() for x in r[:-1] if x is not None]
            ctx.release(pid)
            ctx.release(tid)
            return r
        return f

    def fails(ctx):
        from paper_1101_1245_amd import gpumcd as G
        tid, pid = ctx.load_tables((I.WATER,), I.Physics()), ctx.load_phantom(I.homogeneous((24, 24, 24), 0.5))
        tight = {"queue_items": 64, "secondaries_per_visit": 64, "chunk": 64, "pass_items": 1024}
        with pytest.raises(G.GpumcdError):
            ctx.run_beam(pid, tid, I.Source(I.PHOTON, e=6.0, cx=6, cy=6, wx=4.0, wy=4.0), 20_000, 3, tuning=tight)
        ctx.release(pid)
        ctx.release(tid)
        return []

    return {"big_sparse": one(big, 2000), "small_dense": one(small, 300_000), "big_dense": one(big, 700_000),
            "tally": one(big, 3000, tally=True), "K40": one(small, 5000, K=40), "K1": one(big, 5000, K=1),
            "beams_dev": beams(small, 5, 900, 32, True, True, "torch"), "beams_host": beams(small, 5, 900, 32, True, True, "numpy"),
            "beams_K40": beams(small, 3, 900, 40, True, True, "torch"), "beams_some": beams(small, 6, 900, 32, True, False, None, some=True),
            "beams_plain": beams(big, 3, 2000, 32, False, False, "torch"),
            "beams_few_hist": beams(big, 40, 25, 32, True, False, "torch"),   # fewer than K histories: one-batch slices
            "failed": fails}


def test_jobs_in_any_order_equal_alone():
    from paper_1101_1245_amd import gpumcd as G
    js = jobs()
    alone = {}
    for name, f in js.items():
        with G.Context(0) as c:
            alone[name] = f(c)
    rng = np.random.default_rng(3)
    with G.Context(0) as c:
        for name in list(js) + [str(x) for x in rng.choice(list(js), 40)]:
            for a, b in zip(js[name](c), alone[name]):
                assert np.array_equal(a, b), name
