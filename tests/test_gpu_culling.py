"""Occlusion culling of the visibility matrix, the UE columns and the
validation: scenes whose facets the bounding boxes can go wrong on (tilted,
skewed, without a side, off their plane, far from the origin, more than one
tile of them), every sample count that changes how pairs share a wave.  All
outputs are decisions of the same IEEE FP64 tests as the oracle's and must be
equal."""
import numpy as np
import pytest

import oracle as O
from paper_2301_06399_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2301_06399_amd import mpt
    c = mpt.Context(0)
    yield c
    c.close()


def unit(v):
    return v / np.linalg.norm(v)


def scene(rng, n_planes, n_lines=7, n_quads=4, n_circles=3, offset=0.0, odd=True):
    size = 40.0
    off = np.full(3, offset)
    planes = []
    for i in range(n_planes):
        n = unit(rng.normal(size=3))
        u = unit(np.cross(n, rng.normal(size=3))) * rng.uniform(1, 8)
        v = unit(np.cross(n, u)) * rng.uniform(1, 8)
        o = off + rng.uniform(0, size, 3)
        d = n @ o
        kind = i % 8 if odd else 7
        if kind == 0:
            v = v + 0.4 * u                 # sides not perpendicular
        elif kind == 1:
            u = u + 0.3 * n                 # a side off the plane
        elif kind == 2:
            d = d + 1.5                     # the corner off the plane
        elif kind == 3 and i % 16 == 3:
            v = np.zeros(3)                 # no second side
        planes.append(W.plane_rect(n, d, o, u, v))
    lines = [W.line_seg(off + rng.uniform(0, size, 3), unit(rng.normal(size=3)), 0.0, rng.uniform(1, 9))
             for _ in range(n_lines)]
    quads = [W.paraboloid(off + rng.uniform(0, size, 3), unit(rng.normal(size=3)), rng.uniform(0.5, 2))
             for _ in range(n_quads)]
    if n_quads and odd:
        quads[0][12] = 0.3                  # not a paraboloid of revolution
    circles = [W.circle(off + rng.uniform(0, size, 3), unit(rng.normal(size=3)), rng.uniform(0.5, 2))
               for _ in range(n_circles)]
    return W.Scene(tx=off + rng.uniform(0, size, 3), planes=np.array(planes).reshape(-1, 13),
                   lines=np.array(lines).reshape(-1, 8), quadrics=np.array(quads).reshape(-1, 17),
                   circles=np.array(circles).reshape(-1, 7), aabb_lo=off, aabb_hi=off + size)


@pytest.mark.parametrize("n_planes,k,offset", [(0, 3, 0.0), (1, 1, 0.0), (30, 1, 0.0), (30, 3, 1e5), (33, 7, 0.0),
                                               (20, 9, 0.0), (12, 16, 0.0), (514, 2, 0.0)])
def test_culled_visibility_matches_oracle(ctx, n_planes, k, offset):
    import torch
    from paper_2301_06399_amd import mpt
    rng = np.random.default_rng([n_planes, k])
    sc = scene(rng, n_planes, offset=offset)
    rx = offset + rng.uniform(0, 40, (5, 3))
    rx[1] = sc.tx                            # a segment without a length
    ctx.upload_scene(sc)
    V, B = ctx.visibility(k)
    U, los = ctx.visibility_rx(torch.from_numpy(rx).cuda(), k)
    n = sc.n_prims
    oV, oB = O.visibility(sc, k=k)
    oU, olos = O.visibility_rx(sc, rx, k=k)
    assert np.array_equal(mpt.unpack_bits(V, n), oV)
    assert np.array_equal(mpt.unpack_bits(B, n), oB)
    assert np.array_equal(mpt.unpack_bits(U, n), oU)
    assert np.array_equal(los.cpu().numpy().astype(bool), olos)


@pytest.mark.parametrize("n_planes,n,offset", [(0, 65, 0.0), (40, 3001, 0.0), (40, 500, 1e5), (70, 5000, 0.0)])
def test_culled_validation_matches_oracle(ctx, n_planes, n, offset):
    """Random points as paths: the flags and their count, for a list whose
    length is no multiple of a block."""
    import torch
    from paper_2301_06399_amd import mpt
    rng = np.random.default_rng([n_planes, n, 5])
    sc = scene(rng, n_planes, offset=offset)
    order = rng.integers(1, 6, n).astype(np.int32)
    prim = rng.integers(0, sc.n_prims, (5, n)).astype(np.int32)
    b = W.Batch(offset + rng.uniform(0, 40, (9, 3)), rng.integers(0, 9, n), order, prim)
    # short paths, so that some of them are free
    x = np.zeros((15, n))
    start = b.rx[b.rx_index] + rng.normal(size=(n, 3)) * 3
    for j in range(5):
        x[3 * j:3 * j + 3] = np.where(order > j, (start + rng.normal(size=(n, 3)) * 2).T, 0.0)
    acc = (rng.random(n) < 0.7).astype(np.uint8)
    ctx.upload_scene(sc)
    out = mpt.DeviceOut(n)
    out.x.copy_(torch.from_numpy(mpt.to_rows(x)))
    vis, kept = ctx.visible(mpt.DeviceBatch(b), out, torch.from_numpy(acc).cuda())
    want = O.visible_batch(sc, b, x, acc)
    assert np.array_equal(vis.cpu().numpy(), want)
    assert kept == want.sum()
    assert n_planes == 0 or 0 < want.sum() < acc.sum()


@pytest.mark.parametrize("max_order,edge_last", [(3, 0), (4, 0), (5, 1)])
def test_deep_candidates_match_oracle(ctx, max_order, edge_last):
    """Orders above three (counted by their last objects, then walked) and
    first objects with more successors than the fill's parts."""
    import torch
    from paper_2301_06399_amd import mpt
    rng = np.random.default_rng(max_order)
    n, n_rx = 19 if max_order > 3 else 150, 3
    sc = scene(rng, n - 7, n_lines=4, n_quads=2, n_circles=1, odd=False)
    V = rng.random((n, n)) < (0.35 if max_order > 3 else 0.5)
    V = np.triu(V, 1)
    V = V | V.T
    Bv, U = rng.random(n) < 0.5, rng.random((n_rx, n)) < 0.4
    ctx.upload_scene(sc)

    def words(m):
        w = np.zeros((*m.shape[:-1], (n + 31) // 32 * 32), bool)
        w[..., :n] = m
        return torch.from_numpy(np.packbits(w, axis=-1, bitorder="little").view(np.int32)).cuda()
    rx = np.zeros((n_rx, 3))
    ri, order, prim = ctx.candidates(words(V), words(Bv), words(U), max_order, bool(edge_last))
    want = O.candidates(sc, rx, V, Bv, U, max_order, bool(edge_last))
    assert len(want["order"]) > 100
    assert np.array_equal(ri.cpu().numpy(), want["rx_index"])
    assert np.array_equal(order.cpu().numpy(), want["order"])
    assert np.array_equal(prim.cpu().numpy(), want["prim"])
