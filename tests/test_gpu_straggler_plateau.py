"""Paths parked before or early in their descent keep their plateau test: with
the shortest windows (the test opens every iteration after the first, or every
other) parking changes no output, on batches so small that a wave parks all its
paths before their first pass, and on larger ones."""
import numpy as np
import pytest

from paper_2301_06399_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2301_06399_amd import mpt
    c = mpt.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("prec,form", [(0, 0), (0, 2), (1, 0), (1, 2)])
@pytest.mark.parametrize("win", [1, 2, 3])
def test_parking_keeps_the_plateau_test(ctx, prec, form, win):
    from paper_2301_06399_amd import mpt
    for sc, b in (W.config2(n_rx=128, per_rx=64), W.config3(n_rx=32, per_rx=64)):
        ctx.upload_scene(sc)
        for n in (1, 37, b.n):
            db = mpt.DeviceBatch(b.subset(np.arange(n)))
            for sched in (mpt.SCHED_PERSISTENT, mpt.SCHED_PER_ORDER, mpt.SCHED_SPLIT):
                res = {}
                for spill in (0, 1, 16, 64):
                    out = mpt.DeviceOut(n, stages=True)
                    ctx.solve(db, mpt.default_opts(precision=prec, form=form, plateau_win=win, sched=sched,
                                                   spill=spill), out)
                    res[spill] = out.numpy()
                for spill in (1, 16, 64):
                    for k in ("x", "cost", "iters", "status"):
                        assert np.array_equal(res[spill][k], res[0][k]), (n, sched, spill, k)
            if n == b.n:
                assert (res[0]["iters"] > 1).sum() > n // 10  # the window does not end everything at once


@pytest.mark.parametrize("form", [0, 2])
def test_iterations_of_the_straggler_launch(ctx, form):
    """One wave, 64 lanes, 65 paths: when the first path ends (planar, at its
    cap in the step of iteration 3) the last one is taken and the wave parks
    them all.  The straggler launch runs every iteration of the others after
    the third, and all of the last one's."""
    from paper_2301_06399_amd import mpt
    sc, b = W.config5(n_rx=64)
    ctx.upload_scene(sc)
    opts = dict(form=form, sched=mpt.SCHED_PERSISTENT, max_iter32_planar=3)

    def stages(batch, **more):
        out = mpt.DeviceOut(batch.n, stages=True)
        ctx.solve(mpt.DeviceBatch(batch), mpt.default_opts(**opts, **more), out)
        return out.numpy()["stage"]

    it = stages(b)[0]
    three = b.order == 3
    npl, nln = len(sc.planes), len(sc.lines)
    curved = three & (b.prim[:3] >= npl + nln).any(0)
    planes = three & (b.prim[:3] < npl).all(0)
    capped = np.flatnonzero(planes & (it == 3))
    if len(capped) == 0:                      # lists without a diffraction: made here
        many = b.subset(np.flatnonzero(three))
        rng = np.random.default_rng(2)
        prim = many.prim.copy()
        prim[:3] = rng.integers(0, npl, (3, many.n))
        many.prim = prim
        first = many.subset(np.flatnonzero(stages(many)[0] == 3)[:1])
    else:
        first = b.subset(capped[:1])
    rest = b.subset(np.flatnonzero(curved & (it >= 8))[:64])
    assert first.n == 1 and rest.n == 64
    batch = W.Batch(b.rx, np.concatenate([first.rx_index, rest.rx_index]),
                    np.concatenate([first.order, rest.order]), np.concatenate([first.prim, rest.prim], axis=1))
    st = stages(batch, grid=1, block=64, spill=64, refill=1)
    n, late = st[0], st[3]
    assert n[0] == 3 and late[0] == 0
    left = n[1:] - late[1:]
    assert (left == 3).sum() == 63 and (left == 0).sum() == 1, left
