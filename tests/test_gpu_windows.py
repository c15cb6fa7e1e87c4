"""GPU: the blends' window test and per-lane walks at the edges of a window.

Each wave tests its block's candidates in windows of 32 (none for windows of up to 8) and
every lane then walks its own pixel's share.  Scenes of exactly K surfels whose footprints
all meet one 8 x 8 block, K around the window and batch sizes, so that full, partial and
skipped windows and their remainders all occur; images, contributions, gradients to every
parameter and the pose against the oracle, with the bars of the other parity tests.  The
images are small, so up to 2 % of their pixels may lie within a decision margin (161
surfels of a dozen decisions each, at 1e-5 relative, is 2 % of the pixels)."""

import numpy as np
import pytest
import torch

import oracle
from tests.gpu_common import check_grads, check_images, check_pose, dev, host
from tests.test_gpu_few_surfels import crossing_surfels

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("filt", [True, False])
@pytest.mark.parametrize("k", [1, 8, 9, 31, 32, 33, 64, 65, 128, 129, 161])
def test_window_edges_match_oracle(k, filt):
    from paper_2506_00970_amd import Rasterizer

    params, cam, pose = crossing_surfels(k, seed=k)
    r = Rasterizer(filter=filt)
    out = r.render_batch([(dev(params), cam, dev(pose.reshape(12)))], contribution=True)[0]
    g = np.random.default_rng(1000 + k)
    hw = cam.width * cam.height
    grads = {"d_rgb": g.normal(size=(3, cam.height, cam.width)) / hw, "d_depth": g.normal(size=(cam.height, cam.width)) / hw,
             "d_normal": g.normal(size=(3, cam.height, cam.width)) / hw, "d_alpha": g.normal(size=(cam.height, cam.width)) / hw}
    d = {n: dev(v) for n, v in grads.items()}
    dp, dpose = r.backward_batch(out.generation, [d])[0]
    _, dpose_only = r.backward_batch(out.generation, [d], params_grad=False)[0]
    torch.cuda.synchronize()
    ref = oracle.render(params, cam, pose, filter=filt)
    img = {n: host(getattr(out, n)) for n in ("rgb", "depth", "normal", "alpha")}
    print(k, filt, check_images(img, ref, ref["fmargin"], max_excluded=0.02))
    alpha_sum = img["alpha"].sum()
    assert abs(host(out.contrib).sum() - alpha_sum) <= 1e-4 * max(alpha_sum, 1.0)
    near = ref["gmargin"] < 1e-5
    og = oracle.backward(params, cam, pose, **grads, watch=near, scale=True, scale_mask=near, filter=filt)
    print(check_grads(host(dp), og["d_params"], skip=og["touched"]))
    for p in (dpose, dpose_only):
        check_pose(host(p), og["pose_paper"], scale=og["pose_scale"], flip=og["pose_scale_masked"])
