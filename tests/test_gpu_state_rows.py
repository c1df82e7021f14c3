"""The FP32 pass around the batch size (2^21 solves) above which it keeps its state
rows in a buffer of its own instead of the output rows: a solve's result does not
depend on where its state was, so every output equals that of the same solve in a
small batch, bit for bit, with and without parked stragglers and from a captured
solve."""
import numpy as np
import pytest

from paper_2301_06399_amd import workloads as W

pytestmark = pytest.mark.gpu

LINE = 1 << 21


@pytest.mark.parametrize("n", [LINE, LINE + 1])
@pytest.mark.parametrize("opts", [dict(form=2), dict(form=0, spill=16), dict(form=2, sched=0, spill=16),
                                  dict(form=2, graph=1)], ids=["param", "implicit-parked", "per-order-parked", "graph"])
def test_results_do_not_depend_on_the_state_rows(n, opts):
    import torch
    from paper_2301_06399_amd import mpt
    sc, b = W.config5(n_rx=64)
    order = b.order.copy()
    order[7::1001] = 0                                  # invalid solves
    b.order = order
    ctx = mpt.Context(0)
    try:
        ctx.upload_scene(sc)
        small = ctx.solve(mpt.DeviceBatch(b), mpt.default_opts(form=opts["form"]))
        sel = torch.arange(n, device="cuda") % b.n
        one = mpt.DeviceBatch(b)
        db = mpt.device_batch(one.rx, one.rx_index[sel].contiguous(), one.order[sel].contiguous(),
                              one.prim[:, sel].contiguous())
        out = mpt.DeviceOut(n)
        for rep in range(2):
            out.x.fill_(-1.0)
            out.status.fill_(99)
            ctx.solve(db, mpt.default_opts(**opts), out)
            ctx.synchronize()
            for k in ("cost", "iters", "status", "x"):
                assert torch.equal(getattr(out, k), getattr(small, k)[sel]), (rep, k)
    finally:
        ctx.close()
