"""Which camera renders and batched jobs run in pieces, on both sides of every
limit: a render in pieces takes the stream's work queue, which ends the
validity of a kept render's pieces there, and a one-pass render leaves them, so
that the backward of the kept render runs or is refused."""
import sys

import numpy as np
import pytest

from paper_2103_14024_amd import scenes

pytestmark = pytest.mark.gpu

# depth, degree, index, W, H, options, in pieces
RULE = [
    (7, 1, True, 255, 257, {}, False),
    (7, 1, True, 256, 256, {}, True),
    (7, 1, True, 383, 256, {}, True),
    (7, 1, True, 384, 256, {}, False),
    (7, 4, True, 384, 256, {}, False),
    (3, 1, True, 384, 256, {}, False),
    (3, 1, True, 383, 256, {}, True),
    (8, 2, True, 383, 256, {}, True),
    (8, 2, True, 384, 256, {}, False),
    (8, 4, True, 640, 511, {}, True),
    (8, 4, True, 640, 512, {}, False),
    (8, 2, True, 640, 511, dict(sh_off=2), True),
    (8, 2, True, 640, 512, dict(sh_off=2), False),
    (9, 1, True, 1024, 703, {}, True),
    (9, 1, True, 1024, 704, {}, False),
    (10, 1, True, 2047, 1024, {}, True),
    (10, 1, True, 2048, 1024, {}, False),
    (11, 1, True, 2048, 1024, {}, True),
    (7, 1, False, 383, 256, {}, True),
    (7, 1, False, 384, 256, {}, False),
    (8, 2, False, 768, 767, {}, True),
    (8, 2, False, 768, 768, {}, False),
    (8, 4, False, 640, 511, {}, True),
    (8, 4, False, 640, 512, {}, False),
    (9, 1, False, 1535, 1024, {}, True),
    (9, 1, False, 1536, 1024, {}, False),
    (10, 1, False, 2048, 1024, {}, True),
    (7, 1, True, 1024, 1024, dict(aux=True), True),
    (7, 1, True, 1024, 1024, dict(max_steps=400), True),
    (9, 1, True, 512, 512, dict(one_pass=True), False),
    (9, 1, True, 512, 512, dict(aux=True, one_pass=True), False),
]


@pytest.mark.parametrize("depth,deg,index,W,H,opts,pieces", RULE)
def test_rule(depth, deg, index, W, H, opts, pieces):
    import torch

    import paper_2103_14024_amd as po

    po.reset_device_errors()
    cells = np.array([[depth, 1, 2, 3], [2, 3, 3, 3], [1, 1, 0, 0]], np.int32)
    sig, sh = scenes.leaf_values(3, deg, 5)
    tree = po.Tree.from_cells(depth, deg, cells, sig, sh, index=index)
    cam = po.Camera(scenes.hemisphere_poses(1, 3.0, 3)[0], W, H, *scenes.intrinsics(W, H, 40.0))
    print(f"[gpu] depth {depth}, degree {deg}, index {index}, {W} x {H}, {opts}", file=sys.stderr, flush=True)
    o, d = (torch.from_numpy(a).cuda() for a in scenes.random_rays(64, 3))
    slot = torch.empty(64, dtype=torch.int32, device="cuda")
    gs, gsh = torch.zeros_like(tree.sigma), torch.zeros_like(tree.sh)

    def took_the_queue(render):
        rgb = po.render_rays_keep(tree, o, d, slot)
        render()
        try:
            po.render_rays_backward_kept(tree, o, d, rgb, torch.ones_like(rgb), slot, gs, gsh)
        except po.PlenOctreeError:
            return True
        return False

    assert took_the_queue(lambda: po.render_camera(tree, cam, **opts)) == pieces
    if "max_steps" not in opts:  # jobs count whole tiles
        W16, H16 = (W + 15) // 16 * 16, (H + 15) // 16 * 16
        if W16 * H16 == W * H or not pieces and W * H > 1 << 16:
            job = dict(opts)
            if job.pop("aux", False):
                job["aux_out"] = torch.empty((H, W, 4), device="cuda")
            out = torch.empty((H, W, 3), device="cuda")
            assert took_the_queue(lambda: po.render_batch([po.Job(tree, cam, out, **job)])) == pieces
    assert po.device_errors() == 0
