"""GPU: the depth order of tile lists at the edges of its methods (counted up to 256
entries, merged runs of 64 up to 2048, chunks merged through global memory above), and the
placement of pairs by tile; whole numbers, compared exactly."""

import numpy as np
import pytest
import torch

import synth
from tests.gpu_common import dev

pytestmark = pytest.mark.gpu


def _stack(k, seed):
    """k surfels that all cover the first of four tiles, some all of them, in shuffled
    depth with repeated depths."""
    g = np.random.default_rng(seed)
    cam = synth.Camera(32, 32, 60.0, 60.0, 16.0, 16.0)
    z = g.choice(np.float32(g.uniform(1.0, 4.0, max(k // 3, 1))), k)
    px, py = g.uniform(6.0, 12.0, (2, k))
    mu = np.stack([(px - cam.cx) / cam.fx * z, (py - cam.cy) / cam.fy * z, z])
    tu, tv = np.zeros((3, k)), np.zeros((3, k))
    tu[0], tv[1] = 1.0, 1.0
    s = np.where(g.uniform(size=k) < 0.2, 0.3, 0.01) * np.ones((2, k))
    params = np.concatenate([mu, tu, tv, s, g.uniform(0.01, 0.3, (1, k)), g.uniform(0, 1, (3, k))])
    pose = np.concatenate([np.eye(3), np.zeros((3, 1))], axis=1)
    return params.astype(np.float32), cam, pose.astype(np.float32)


@pytest.mark.parametrize("k", [1, 2, 63, 64, 65, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049,
                               4096, 4097, 10001])
def test_tile_list_order(k):
    from paper_2506_00970_amd import Rasterizer

    params, cam, pose = _stack(k, seed=k)
    r = Rasterizer(keep_unsorted=True)
    for _ in range(2):  # (the second render finds the first one's counters and buffers)
        r.render(dev(params), cam, dev(pose.reshape(12)))
        torch.cuda.synchronize()
        c = r.counts()
        assert c["overflow"] == 0 and c["n_visible"] == k
        ukeys, uids, dk = r.debug("unsorted_keys"), r.debug("unsorted_ids"), r.debug("depth_keys")
        order = np.lexsort((uids, dk[uids], ukeys))
        np.testing.assert_array_equal(r.debug("tile_keys"), ukeys[order])
        np.testing.assert_array_equal(r.debug("tile_ids"), uids[order])
        rng = r.debug("ranges").reshape(-1, 2).astype(np.int64)
        np.testing.assert_array_equal(rng[:, 1] - rng[:, 0], np.bincount(ukeys, minlength=4))
        assert rng[0, 1] - rng[0, 0] == k
