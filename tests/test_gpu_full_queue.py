"""Renders and gradients in pieces whose work queue fills up: a rod of fog of
1024 x 16 x 16 finest cells along the box, seen end on, so that every ray wants
all of its 16 pieces, and every piece all of its sub-pieces, at both levels of
the queue.  262,144 rays ask for four times the pieces it holds (and eight
times of the fixed queue's); those that find their region full are finished by
their own lane.  Against the one-pass kernels and the FP64 oracle, for samples
shaded by their own lane, by quads and through the wave's queue."""
import sys

import gradcheck
import numpy as np
import oracle
import pytest

from paper_2103_14024_amd import scenes

pytestmark = pytest.mark.gpu
TOL = 1e-4
SLOTS = 1 << 20  # of a level of the queue


def _rod(deg):
    n, w = 1 << 10, 16
    a = np.arange((n - w) // 2, (n + w) // 2)
    x, y, z = np.meshgrid(np.arange(n), a, a, indexing="ij")
    ijk = np.column_stack([x.ravel(), y.ravel(), z.ravel()])
    cells = np.column_stack([np.full(len(ijk), 10), ijk]).astype(np.int32)
    _, sh = scenes.leaf_values(len(cells), deg, 6)
    # opaque along about two thirds of the rod
    sig = np.random.default_rng(7).uniform(4.0, 10.0, len(cells)).astype(np.float32)
    return dict(depth=10, sh_degree=deg, center=(0.0, 0.0, 0.0), half=1.0, cells=cells, sigma=sig, sh=sh)


def _rays(n, seed):
    """Through both ends of the rod."""
    rng = np.random.default_rng(seed)
    p, q = rng.uniform(-0.014, 0.014, (2, n, 2))
    end = rng.choice([-1.0, 1.0], n)
    a, b = np.column_stack([-end, p]), np.column_stack([end, q])
    return (a - 0.7 * (b - a)).astype(np.float32), (b - a).astype(np.float32)


def _check(got, one, want, idx, stop_T):
    assert float((got - one).abs().max()) <= TOL + stop_T
    # (a T within rounding of stop_T may stop one sample apart: stop_T of weight)
    assert np.abs(got.reshape(-1, 3)[idx].cpu().numpy() - want).max() <= TOL + stop_T


@pytest.mark.parametrize("stop_T", [0.0, 1e-4])
@pytest.mark.parametrize("deg,index", [(1, True), (3, True), (4, True), (3, False)])
def test_camera(deg, index, stop_T):
    import torch

    import paper_2103_14024_amd as po

    po.reset_device_errors()
    s, W = _rod(deg), 512
    tree = po.Tree.from_scene(s, index=index)
    f = 0.5 * W / 0.0035
    pose = scenes.look_at(np.array([3.0, 1e-4, 2e-4]), (0.0, 0.0, 0.0))
    cam = po.Camera(pose, W, W, f, f, 0.5 * W, 0.5 * W)
    print(f"[gpu] K = {(deg + 1) ** 2}, index {index}, stop_T {stop_T}", file=sys.stderr, flush=True)
    _, aux = po.render_camera(tree, cam, stop_T=0.0, aux=True, one_pass=True)
    # 16 pieces of at least 60 samples each: handed on again past 24
    assert float(aux[..., 1].min()) > 1000 and 16 * W * W >= 4 * SLOTS
    one = po.render_camera(tree, cam, stop_T=stop_T, one_pass=True)
    f32 = float(np.float32(f))
    o, d = oracle.camera_rays(np.asarray(pose, np.float32).astype(np.float64), W, W, f32, f32, 0.5 * W, 0.5 * W)
    idx = np.random.default_rng(3).choice(W * W, 400, replace=False)
    ot = oracle.OracleTree(s["depth"], deg, s["center"], s["half"], s["cells"], s["sigma"], s["sh"])
    want = ot.render_rays(o[idx], d[idx], gamma=stop_T)[0]
    _check(po.render_camera(tree, cam, stop_T=stop_T), one, want, idx, stop_T)
    _check(po.render_camera(tree, cam, stop_T=stop_T, aux=True)[0], one, want, idx, stop_T)
    out = torch.empty_like(one)
    po.render_camera_noalloc(tree, cam, out, stop_T=stop_T)
    _check(out, one, want, idx, stop_T)
    assert po.device_errors() == 0


@pytest.mark.parametrize("n", [200000, 300000])
@pytest.mark.parametrize("deg,index", [(1, True), (3, True), (4, True), (1, False)])
def test_list_and_gradients(deg, index, n):
    import torch

    import paper_2103_14024_amd as po

    po.reset_device_errors()
    s = _rod(deg)
    tree = po.Tree.from_scene(s, index=index)
    o, d = _rays(n, 5)
    og, dg = torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda()
    print(f"[gpu] K = {(deg + 1) ** 2}, index {index}, {n} rays", file=sys.stderr, flush=True)
    idx = np.random.default_rng(3).choice(n, 400, replace=False)
    ot = oracle.OracleTree(s["depth"], deg, s["center"], s["half"], s["cells"], s["sigma"], s["sh"])
    slot = torch.empty(n, dtype=torch.int32, device="cuda")
    for stop_T in (1e-4, 0.0):
        one = po.render_rays(tree, og, dg, stop_T=stop_T, one_pass=True)
        want = ot.render_rays(o[idx], d[idx], gamma=stop_T)[0]
        _check(po.render_rays(tree, og, dg, stop_T=stop_T), one, want, idx, stop_T)
        kept = po.render_rays_keep(tree, og, dg, slot, stop_T=stop_T)
        _check(kept, one, want, idx, stop_T)
    # every ray has cells left after the first walk: those without a slot found their region full
    assert int((slot >= 0).sum()) > 1000 and int((slot < 0).sum()) > n // 2
    g = torch.from_numpy(np.random.default_rng(9).standard_normal((n, 3)).astype(np.float32)).cuda()
    ks, ksh = torch.zeros_like(tree.sigma), torch.zeros_like(tree.sh)
    po.render_rays_backward_kept(tree, og, dg, kept, g, slot, ks, ksh, stop_T=0.0)
    gs, gsh = po.render_rays_backward(tree, og, dg, kept, g, stop_T=0.0)
    hs, hsh = po.render_rays_backward(tree, og, dg, one, g, stop_T=0.0, one_pass=True)
    for name, (a, b) in (("kept", (ks, ksh)), ("split", (gs, gsh))):
        for x, y, what in ((a, hs, "dsigma"), (b, hsh, "dsh")):
            y = y.double().cpu().numpy()
            gradcheck.check(x.cpu().numpy(), y, y, f"{name} {what}")
    assert po.device_errors() == 0
