"""One batch over trees of every kind of walk: indexed with the grid at the
bricks, indexed with nodes between, and the caller's child array.  Every job's
pixels equal those of its own render bit for bit, in a mixed launch and in one
of a single kind, for records shaded by their own lane, by quads and through
the queue."""
import sys

import numpy as np
import pytest

from paper_2103_14024_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("deg", [1, 3, 4])
def test_mixed_batch(deg, dtype):
    import torch

    import paper_2103_14024_amd as po

    po.reset_device_errors()
    trees = []
    for depth, level, index in ((6, 6, True), (3, 3, True), (12, 5, True), (6, 6, False), (12, 5, False)):
        cells = scenes.random_tree_cells(level, depth)
        if depth > level:  # some leaves of the finest level instead of a coarse one
            lv, i, j, k = cells[0]
            up = 1 << (depth - lv)
            fine = np.array([i, j, k]) * up + np.array([[0, 0, 0], [1, 0, 1], [up - 1, up // 2, up - 1]])
            cells = np.concatenate([cells[1:], np.column_stack([np.full(3, depth), fine])]).astype(np.int32)
        sig, sh = scenes.leaf_values(len(cells), deg, 5)
        trees.append(po.Tree.from_cells(depth, deg, cells, sig, sh, dtype=dtype, index=index))
    print(f"[gpu] degree {deg}, {dtype}: leaves {[t.n_leaves for t in trees]}", file=sys.stderr, flush=True)
    sizes = [(64, 48), (33, 70), (17, 16), (90, 31), (48, 48)]
    cams = [po.Camera(scenes.hemisphere_poses(1, 3.0, 3 + i)[0], W, H, *scenes.intrinsics(W, H, 45.0))
            for i, (W, H) in enumerate(sizes)]
    own = [po.render_camera(t, c) for t, c in zip(trees, cams)]
    assert all(float((o - 1.0).abs().max()) > 0.05 for o in own)
    for pick in ([0, 1, 2, 3, 4], [2, 0], [3, 1], [2, 4], [0, 0]):
        outs = [torch.full_like(own[i], -1.0) for i in pick]
        po.render_batch([po.Job(trees[i], cams[i], o) for i, o in zip(pick, outs)])
        for i, o in zip(pick, outs):
            assert torch.equal(o, own[i]), (pick, i)
    assert po.device_errors() == 0
