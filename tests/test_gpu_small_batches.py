"""Batches at the sizes where the binning (16,384 solves) and the acceptance
(262,144) change their launches, invalid solves among them.  A solve's result
does not depend on the batch it is in, so every output has to equal that of
the same solve in the larger batch, bit for bit."""
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


def run(ctx, b, stages, **opts):
    import torch
    from paper_2301_06399_amd import mpt
    db = mpt.DeviceBatch(b)
    out = mpt.DeviceOut(b.n, stages=stages)
    for t in (out.x, out.cost, out.iters, out.status):
        t.fill_(77)
    ctx.solve(db, mpt.default_opts(**opts), out)
    acc, idx, k = ctx.accept(db, out)
    r = out.numpy()
    r["accept"] = acc.cpu().numpy()
    assert k == int(r["accept"].sum())
    assert np.array_equal(idx.cpu().numpy(), np.flatnonzero(r["accept"]))
    return r


def batch(config):
    sc, b = config(n_rx=300, per_rx=64)
    b = b.subset(np.arange(16385))
    order, prim, rxi = b.order.copy(), b.prim.copy(), b.rx_index.copy()
    order[5::97] = 0
    order[11::97] = 6
    prim[0, 17::97] = 1 << 20
    rxi[23::97] = -1
    b.order, b.prim, b.rx_index = order, prim, rxi
    return sc, b


@pytest.mark.parametrize("config,opts", [(W.config2, dict()), (W.config2, dict(precision=0)),
                                         (W.config6, dict()), (W.config3, dict())],
                         ids=["street", "street-fp64", "glazed", "curved"])
def test_results_do_not_depend_on_the_batch(ctx, config, opts):
    sc, b = batch(config)
    ctx.upload_scene(sc)
    full = run(ctx, b, True, **opts)
    assert (full["status"] == 5).sum() > 16385 // 97 and full["accept"].sum() > 100
    rng = np.random.default_rng(1)
    for n in (1, 2, 63, 255, 257, 1024, 1025, 4095, 4097, 16383, 16384):
        sel = rng.permutation(b.n)[:n]
        g = run(ctx, b.subset(sel), n % 2 == 1, **opts)
        for key in ("cost", "iters", "status", "accept"):
            assert np.array_equal(g[key], full[key][sel]), (n, key)
        assert np.array_equal(g["x"], full["x"][:, sel]), n
        if n % 2:
            assert np.array_equal(g["stage"], full["stage"][:, sel]), n


@pytest.mark.parametrize("n", [262144, 262145])
def test_acceptance_around_the_list(ctx, n):
    sc, b = batch(W.config2)
    ctx.upload_scene(sc)
    full = run(ctx, b, False)
    sel = np.arange(n) % b.n
    g = run(ctx, b.subset(sel), False)
    assert np.array_equal(g["accept"], full["accept"][sel])
