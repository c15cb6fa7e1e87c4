"""GPU: gradients of views with fewer surfels than a pose has entries.

The backward reads the pose as the render kept it, all twelve entries also when the view
has only one surfel."""

import numpy as np
import pytest
import torch

import oracle
import synth
from tests.gpu_common import check_grads, check_pose, dev, host

pytestmark = pytest.mark.gpu


def crossing_surfels(k, seed):
    """k small tilted surfels whose projected centres lie in the block [8, 15] x [8, 15]."""
    g = np.random.default_rng(seed)
    cam = synth.Camera(27, 21, 40.0, 40.0, 13.0, 10.0)
    z = g.uniform(1.5, 3.0, k)
    px, py = g.uniform(8.5, 14.5, (2, k))
    mu = np.stack([(px - cam.cx) / cam.fx * z, (py - cam.cy) / cam.fy * z, z])
    tu, tv = g.normal(size=(2, 3, k)) * [[[1.0], [1.0], [0.4]]]
    tu /= np.linalg.norm(tu, axis=0)
    tv -= (tu * tv).sum(axis=0) * tu
    tv /= np.linalg.norm(tv, axis=0)
    s = np.exp(g.uniform(np.log(0.01), np.log(0.12), (2, k)))
    params = np.concatenate([mu, tu, tv, s, g.uniform(0.02, 0.25, (1, k)), g.uniform(0, 1, (3, k))])
    pose = np.concatenate([np.eye(3), np.zeros((3, 1))], axis=1)
    return params.astype(np.float32), cam, pose.astype(np.float32)


@pytest.mark.parametrize("n", [1, 2, 5, 11, 12, 13])
def test_gradients_of_few_surfels(n):
    from paper_2506_00970_amd import Rasterizer

    params, cam, pose = crossing_surfels(n, seed=100 + n)
    r = Rasterizer()
    out = r.render(dev(params), cam, dev(pose.reshape(12)))
    g = np.random.default_rng(n)
    hw = cam.width * cam.height
    grads = {"d_rgb": g.normal(size=(3, cam.height, cam.width)) / hw, "d_depth": g.normal(size=(cam.height, cam.width)) / hw}
    dp, dpose = r.backward(out.generation, **{k: dev(v) for k, v in grads.items()})
    torch.cuda.synchronize()
    near = oracle.render(params, cam, pose)["gmargin"] < 1e-5
    og = oracle.backward(params, cam, pose, **grads, watch=near, scale=True, scale_mask=near)
    check_grads(host(dp), og["d_params"], skip=og["touched"])
    check_pose(host(dpose), og["pose_paper"], scale=og["pose_scale"], flip=og["pose_scale_masked"])
