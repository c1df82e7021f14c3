"""Candidate enumeration at object counts around the words and waves that hold a
row of the visibility matrix (32 objects a word, 64 words a wave), with rows
whose paths have nothing to write and enough receivers that a first object is
split or not.  The expected lists are enumerated on the CPU from the same bits;
they are whole numbers and must be equal."""
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


def words(rows):
    rows = np.atleast_2d(rows)
    w = np.zeros((rows.shape[0], (rows.shape[1] + 31) // 32), np.uint32)
    for r, c in zip(*np.nonzero(rows)):
        w[r, c // 32] |= np.uint32(1 << (c % 32))
    return w.view(np.int32)


def enumerate_paths(V, B, U, max_order):
    succ = [np.flatnonzero(r) for r in V]
    out = []
    for r in range(U.shape[0]):
        for order in range(1, max_order + 1):
            def walk(path):
                if len(path) == order:
                    if U[r, path[-1]]:
                        out.append((r, order, tuple(path)))
                    return
                for v in succ[path[-1]]:
                    if v not in path:
                        walk(path + [int(v)])
            for v in np.flatnonzero(B):
                walk([int(v)])
    return out


@pytest.mark.parametrize("n,n_rx,max_order", [(31, 2, 3), (64, 40, 3), (65, 3, 4), (2047, 1, 3), (2049, 2, 3),
                                              (2113, 3, 4), (4096, 1, 3)])
def test_lists_around_the_words(ctx, n, n_rx, max_order):
    import torch
    rng = np.random.default_rng(n)
    lines = [W.line_seg(rng.uniform(0, 50, 3), np.array([0.0, 0.0, 1.0]), 0.0, 1.0) for _ in range(n)]
    ctx.upload_scene(W.Scene(tx=np.array([25.0, 25.0, 20.0]), planes=np.zeros((0, 13)), lines=np.array(lines),
                             aabb_lo=np.zeros(3), aabb_hi=np.full(3, 50.0)))
    V = np.zeros((n, n), bool)
    for i in range(n):
        V[i, rng.integers(0, n, 6)] = True
    V[:, n - 1] = rng.random(n) < 0.3            # the last bit of the last word
    V[np.arange(n), np.arange(n)] = False
    B = rng.random(n) < 5.0 / n
    B[[0, n - 1]] = True
    V[n - 1, rng.integers(0, n - 1, min(n - 1, 300))] = True   # more successors than a block has threads
    U = rng.random((n_rx, n)) < 0.4
    U[:, n - 1] = True
    U[-1] = False                                  # a receiver that sees nothing
    dev = [torch.from_numpy(np.ascontiguousarray(words(x))).cuda() for x in (V, B, U)]
    ri, order, prim = ctx.candidates(dev[0], dev[1].reshape(-1), dev[2], max_order)
    want = enumerate_paths(V, B, U, max_order)
    assert len(want) == ri.numel()
    got = list(zip(ri.cpu().tolist(), order.cpu().tolist(), prim.cpu().numpy().T.tolist()))
    for (r, o, p), (gr, go, gp) in zip(want, got):
        assert (r, o, list(p) + [-1] * (5 - o)) == (gr, go, gp)
