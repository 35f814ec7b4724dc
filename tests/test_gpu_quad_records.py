"""Float32 records of 16 coefficients, loaded by quads of lanes, where a wave's
lanes differ most: absent lanes, rays that miss next to rays that hit, early
stops, trees without a grid or an index.  Colours against the FP64 oracle at
the render's bar."""
import sys

import numpy as np
import oracle
import pytest

from paper_2103_14024_amd import scenes

pytestmark = pytest.mark.gpu
TOL = 1e-4


@pytest.mark.parametrize("stop_T", [0.0, 1e-2])
@pytest.mark.parametrize("depth,index", [(2, True), (5, True), (5, False)])
@pytest.mark.parametrize("n", [1, 3, 63, 66, 197])
def test_quad_render(n, depth, index, stop_T):
    import torch

    import paper_2103_14024_amd as po

    po.reset_device_errors()
    c = (np.arange(1 << depth) + 0.5) * (2.0 / (1 << depth)) - 1.0
    x, y, z = np.meshgrid(c, c, c, indexing="ij")
    ijk = np.argwhere(x * x + y * y + z * z <= 0.64)
    cells = np.column_stack([np.full(len(ijk), depth), ijk]).astype(np.int32)
    _, sh = scenes.leaf_values(len(cells), 3, 6)
    sig = np.random.default_rng(8).uniform(1.0, 6.0, len(cells)).astype(np.float32)
    sig[::7] = -1.0
    o, d = scenes.random_rays(n, 300 + n, radius=2.5, spread=0.6)
    d[1::3] = -d[1::3]  # misses, at every place of a quad
    print(f"[gpu] K = 16, depth {depth}, index {index}, {n} rays, stop_T {stop_T}", file=sys.stderr, flush=True)
    ot = oracle.OracleTree(depth, 3, (0.0, 0.0, 0.0), 1.0, cells, sig, sh)
    o64, d64 = o.astype(np.float64), d.astype(np.float64)
    want = ot.render_rays(o64, d64, gamma=stop_T)[0]
    # (a T within rounding of stop_T may stop one sample apart: stop_T of weight)
    bar = np.full(n, TOL)
    near = ot.render_rays(o64, d64, gamma=stop_T * (1 + 1e-5))[2] != \
        ot.render_rays(o64, d64, gamma=stop_T * (1 - 1e-5))[2]
    bar[near] += stop_T
    tree = po.Tree.from_cells(depth, 3, cells, sig, sh, index=index)
    og, dg = torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda()
    got, aux = po.render_rays(tree, og, dg, stop_T=stop_T, aux=True)
    assert (np.abs(got.cpu().numpy() - want).max(1) <= bar).all()
    assert torch.equal(got, po.render_rays(tree, og, dg, stop_T=stop_T))
    assert (aux[1::3, 1:3] == 0).all()  # the misses: no sample, no cell
    assert po.device_errors() == 0
