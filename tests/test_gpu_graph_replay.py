"""A captured solve (graph=1) does not outlive what it was captured with.  Its
kernels hold the addresses of the context's workspace, so a direct solve in
between that needs a larger one (another precision, more solves, the learned
start) has to lead to a new capture: the outputs equal those of the direct
solve bit for bit, and memory that has been given out meanwhile keeps its
values."""
import numpy as np
import pytest

from paper_2301_06399_amd import workloads as W

pytestmark = pytest.mark.gpu

KEYS = ("x", "cost", "iters", "status")


def same(got, want):
    return all(np.array_equal(got[k], want[k], equal_nan=True) for k in KEYS)


def curved():
    return W.config3(n_rx=64, per_rx=64)


@pytest.mark.parametrize("graph,between,grow", [
    (dict(precision=0), dict(precision=1), 1),            # FP32 state rows where FP64 had a few lists
    (dict(precision=0, spill=16), dict(precision=1), 1),  # parked FP64 state behind those lists
    (dict(precision=1), dict(precision=1), 4),            # more solves
    (dict(precision=0), dict(precision=0), 5),
    (dict(precision=1, init=2), dict(precision=1, init=2), 4),   # learned start points as well
], ids=["fp32-between", "fp32-between-stragglers", "larger", "larger-fp64", "larger-learned"])
def test_replay_after_the_workspace_grew(graph, between, grow):
    import torch
    from paper_2301_06399_amd import mpt
    assert mpt.INIT_LEARNED == 2
    sc, b = curved()
    ctx, ref_ctx = mpt.Context(0), mpt.Context(0)
    try:
        for c in (ctx, ref_ctx):
            c.upload_scene(sc)
            c.mlp_init(5)
        db = mpt.DeviceBatch(b)
        big = mpt.DeviceBatch(b.subset(np.tile(np.arange(b.n), grow)))
        want = ref_ctx.solve(db, mpt.default_opts(**graph)).numpy()
        out = mpt.DeviceOut(b.n)
        for rep in range(3):
            out.x.fill_(-1.0)
            out.status.fill_(99)
            ctx.solve(db, mpt.default_opts(graph=1, **graph), out)
            ctx.synchronize()
            assert same(out.numpy(), want), rep
            if rep == 0:
                ctx.solve(big, mpt.default_opts(**between))
                ctx.synchronize()
                keep = [torch.full((1 << 18,), 7, dtype=torch.int32, device="cuda") for _ in range(8)]
                torch.cuda.synchronize()
        assert all(bool((k == 7).all()) for k in keep)
    finally:
        ctx.close()
        ref_ctx.close()


@pytest.mark.parametrize("prec,form", [(1, 2), (1, 0), (0, 2)])
def test_replay_after_facets_start_to_refract(prec, form):
    """The same geometry uploaded with and without refractive indices: the
    scene's buffers and sizes stay, the kernels of the solve do not."""
    import dataclasses
    from paper_2301_06399_amd import mpt
    glass, b = W.config6(n_rx=64)
    mirrors = dataclasses.replace(glass, refraction=np.zeros((0, 2)))
    db = mpt.DeviceBatch(b)
    want = []
    for sc in (mirrors, glass):
        ref = mpt.Context(0)
        ref.upload_scene(sc)
        want.append(ref.solve(db, mpt.default_opts(precision=prec, form=form)).numpy())
        ref.close()
    assert not same(want[0], want[1])
    ctx = mpt.Context(0)
    out = mpt.DeviceOut(b.n)
    for rep in range(4):
        ctx.upload_scene((mirrors, glass)[rep % 2])
        for again in range(2):
            out.x.fill_(-1.0)
            out.status.fill_(99)
            ctx.solve(db, mpt.default_opts(precision=prec, form=form, graph=1), out)
            ctx.synchronize()
            assert same(out.numpy(), want[rep % 2]), (rep, again)
    ctx.close()


@pytest.mark.parametrize("sched", ["SCHED_PER_ORDER", "SCHED_SPLIT", "SCHED_PERSISTENT"])
def test_capture_behind_launches_side_by_side(sched):
    """A solve is captured on one of the streams that direct solves launch on:
    captured while such launches are still queued, in every schedule, it gives
    the direct solve's results, and so do they."""
    from paper_2301_06399_amd import mpt
    sc, b = curved()
    ctx = mpt.Context(0)
    try:
        ctx.upload_scene(sc)
        db = mpt.DeviceBatch(b)
        large = mpt.DeviceBatch(b.subset(np.tile(np.arange(b.n), 8)))
        opts = dict(sched=getattr(mpt, sched), form=2)
        want = ctx.solve(db, mpt.default_opts(**opts)).numpy()
        many = ctx.solve(large, mpt.default_opts(**opts)).numpy()
        queued = [mpt.DeviceOut(large.n) for _ in range(3)]
        out = [mpt.DeviceOut(b.n) for _ in range(3)]
        for q, o in zip(queued, out):
            ctx.solve(large, mpt.default_opts(sched=mpt.SCHED_PER_ORDER, form=2), q)
            ctx.solve(db, mpt.default_opts(graph=1, **opts), o)   # new outputs: a new capture
            ctx.solve(db, mpt.default_opts(graph=1, **opts), o)
        for q, o in zip(queued, out):
            assert same(o.numpy(), want) and same(q.numpy(), many)
    finally:
        ctx.close()
