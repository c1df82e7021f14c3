"""The FP32 implicit solver at the batch sizes where its launch changes (one wave
on a CU, two, one per SIMD; side by side each launch by its own paths).  How a
batch is spread over waves changes no result: every output has to equal that of
blocks of 256, bit for bit."""
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


@pytest.mark.parametrize("config,scheds", [(W.config3, ("SCHED_PERSISTENT", "SCHED_PER_ORDER", "SCHED_SPLIT")),
                                           (W.config6, ("SCHED_PERSISTENT",))], ids=["curved", "glazed"])
def test_launch_sizes(ctx, config, scheds):
    import torch
    from paper_2301_06399_amd import mpt
    lanes = torch.cuda.get_device_properties(0).multi_processor_count * 64
    sc, b = config(n_rx=2 * lanes // 64 + 1, per_rx=64)
    ctx.upload_scene(sc)
    tile = np.arange(8 * lanes + 4) % b.n
    for name in scheds:
        sched = getattr(mpt, name)
        if sched == mpt.SCHED_PERSISTENT:
            sizes = ((63, 64), (lanes, 64), (lanes + 1, 64), (2 * lanes, 64), (2 * lanes + 1, 256))
        else:
            sizes = ((63, 256), (lanes // 8, 256), (lanes // 8 + 1, 64), (5 * lanes, 64), (8 * lanes, 64),
                     (8 * lanes + 1, 256))
        for n, block in sizes:
            db = mpt.DeviceBatch(b.subset(tile[:n]))
            res = []
            for blk in (0, 256):
                out = mpt.DeviceOut(n)
                ctx.solve(db, mpt.default_opts(form=0, sched=sched, block=blk), out)
                if not blk:
                    assert ctx.last_launch()["block"] == block, (name, n)
                res.append(out.numpy())
            for k in ("x", "cost", "iters", "status"):
                assert np.array_equal(res[0][k], res[1][k]), (name, n, k)


def test_one_order_takes_the_whole_launch(ctx):
    """Launches side by side with every path in one of them."""
    from paper_2301_06399_amd import mpt
    sc, b = W.config3(n_rx=512, per_rx=64)
    ctx.upload_scene(sc)
    for order in (2, 4, 5):
        few = np.flatnonzero(b.order == order)
        for n in (3000, 17000, 40000):
            db = mpt.DeviceBatch(b.subset(few[np.arange(n) % len(few)]))
            res = [ctx.solve(db, mpt.default_opts(form=0, sched=mpt.SCHED_PER_ORDER, block=blk)).numpy()
                   for blk in (0, 256)]
            assert all(np.array_equal(res[0][k], res[1][k]) for k in ("x", "cost", "iters", "status")), (order, n)
