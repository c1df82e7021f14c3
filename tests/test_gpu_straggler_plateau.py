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
