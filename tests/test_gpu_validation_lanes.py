"""Validation with four lanes or a whole wave to a path: numbers of occluders and
of kept paths at the edges of both, lists at the edges of a wave's and a block's
paths.  The flags are the oracle's decisions and must be equal."""
import numpy as np
import pytest

import oracle as O
from paper_2301_06399_amd import workloads as W
from test_gpu_culling import scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2301_06399_amd import mpt
    c = mpt.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n_planes,n_quads", [(0, 0), (1, 0), (0, 3), (2, 2), (3, 2), (92, 4), (96, 0), (93, 4),
                                              (97, 0)])
def test_lanes_of_a_path(ctx, n_planes, n_quads):
    import torch
    from paper_2301_06399_amd import mpt
    rng = np.random.default_rng([n_planes, n_quads, 7])
    sc = scene(rng, n_planes, n_quads=n_quads)
    ctx.upload_scene(sc)
    # kept paths up to which each gets a wave
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    line = (n_planes + n_quads) * cus * 32 // 20
    for n in (1, 15, 17, 63, 65, 257, 4099, line + 50, line + 51):
        order = rng.integers(1, 6, n).astype(np.int32)
        prim = rng.integers(0, sc.n_prims, (5, n)).astype(np.int32)
        b = W.Batch(rng.uniform(0, 40, (9, 3)), rng.integers(0, 9, n), order, prim)
        x = np.zeros((15, n))
        start = b.rx[b.rx_index] + rng.normal(size=(n, 3)) * 3
        for j in range(5):
            x[3 * j:3 * j + 3] = np.where(order > j, (start + rng.normal(size=(n, 3)) * 2).T, 0.0)
        keep = n - 50 if n >= line + 50 and n > 4099 else int(0.7 * n) + 1
        acc = np.zeros(n, np.uint8)
        acc[rng.permutation(n)[:keep]] = 1
        out = mpt.DeviceOut(n)
        out.x.copy_(torch.from_numpy(mpt.to_rows(x)))
        vis, kept = ctx.visible(mpt.DeviceBatch(b), out, torch.from_numpy(acc).cuda())
        want = O.visible_batch(sc, b, x, acc)
        assert np.array_equal(vis.cpu().numpy(), want), n
        assert kept == want.sum()
    assert 0 < want.sum() <= acc.sum()
