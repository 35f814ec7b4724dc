"""Measured work of the renderer: single calls through its public entry points.

The scenes are those of the repository's own benchmark and tests: the surface
band of a sum of 20 Gaussian blobs (two voxels each side of an iso-surface;
2.9M leaves at depth 9, 0.64M at depth 8) and the shell of three spheres
(2,090 leaves at depth 5), raw densities ~ lognormal(2, 1) and basis
coefficients ~ N(0, 0.5^2), cameras on the upper hemisphere of radius 4 with a
40 degree field of view, white background, early stop below 1e-4.  A seed
draws the leaf values, the poses, the rays, the targets and the incoming
gradients; the geometry of a scene is part of the case.

`exact` walks the same rays in float64 with torch alone, on a dense grid of
leaf numbers.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2103_14024_amd as po
from paper_2103_14024_amd.optim import Trainer
from paper_2103_14024_amd.visibility import leaf_weights

DEV = "cuda"
STOP_T = 1e-4


# ------------------------------------------------------------------- the cases

def listed():
    return [
        # the smallest call: a thumbnail of a small scene, where the launch and
        # one walk's latency count
        dict(name="thumb_64_f32", kind="view", scene="spheres", depth=5, degree=2, leaf="f32", W=64, H=64),
        # a small preview of a served scene, ragged size, one-pass render
        dict(name="preview_243x187_f16", kind="view", scene="blobs", geom=11, depth=8, degree=2, leaf="f16", W=243,
             H=187),
        # the benchmark frame: 512^3 finest grid, degree-3 SH, float32 leaves
        dict(name="frame_800_f32", kind="view", scene="blobs", geom=0, depth=9, degree=3, leaf="f32", W=800, H=800),
        # the largest frame served, float16 leaves
        dict(name="frame_1080p_f16", kind="view", scene="blobs", geom=0, depth=9, degree=3, leaf="f16", W=1920, H=1080),
        # interactive viewer: depth and alpha, two SH bands, a slicing plane
        dict(name="viewer_512_f32", kind="viewer", scene="blobs", geom=12, depth=8, degree=2, leaf="f32", W=512, H=512,
             sh_off=480, clip=True),
        # spherical-Gaussian basis of 25 lobes
        dict(name="sg25_400_f32", kind="view", scene="blobs", geom=1, depth=8, degree=4, leaf="sg", W=400, H=400),
        # compressed leaves: 16-bit positions in per-basis codebooks
        dict(name="codebook_640x480", kind="view", scene="blobs", geom=1, depth=8, degree=3, leaf="codebook", W=640,
             H=480),
        # a free ray list, ragged and below the size that is cut into pieces
        dict(name="rays_30001_f32", kind="rays", scene="blobs", geom=1, depth=8, degree=2, leaf="f32", n=30001),
        # gradient of a small batch through autograd
        dict(name="grad_8191_f32", kind="grad", scene="blobs", geom=3, depth=7, degree=2, leaf="f32", n=8191),
        # one optimisation step of the octree fit
        dict(name="train_65536_f32", kind="train", scene="blobs", geom=1, depth=8, degree=2, leaf="f32", n=65536),
        # one view of the visibility filter of the conversion
        dict(name="filter_800_f32", kind="filter", scene="blobs", geom=0, depth=9, degree=1, leaf="f32", W=800, H=800),
        # one serving launch: chunks of small requests over two resident scenes
        dict(name="batch_6_f16", kind="batch", scene="blobs", geom=11, depth=8, degree=2, leaf="f16", jobs=6, W=256,
             H=256),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["view"] * 5 + ["viewer", "rays", "rays", "grad", "grad", "train", "train", "filter", "batch"])
    c = dict(kind=kind, scene="blobs", geom=rng.choice([0, 1, 3, 11, 12]), depth=rng.choice([6, 7, 8, 8, 9]),
             degree=rng.choice([1, 2, 2, 3, 3]), leaf="f32")
    if kind in ("view", "viewer", "filter"):
        c["W"], c["H"] = _log(rng, 50, 1200), _log(rng, 50, 800)
    if kind in ("view", "rays"):
        c["leaf"] = rng.choice(["f32", "f32", "f16", "f16", "codebook", "sg"])
    if kind == "viewer":
        c["sh_off"], c["clip"] = rng.choice([0, 0, 14, 480]), rng.random() < 0.5
    if kind == "rays":
        c["n"] = _log(rng, 300, 400000)
    if kind == "grad":
        c["n"] = _log(rng, 500, 100000)
    if kind == "train":
        c["depth"], c["n"] = rng.choice([7, 8]), _log(rng, 2000, 150000)
    if kind == "batch":
        c["leaf"], c["jobs"] = "f16", rng.randint(2, 16)
        c["W"], c["H"] = _log(rng, 40, 260), _log(rng, 40, 260)
    return c


# -------------------------------------------------------------- scene geometry

_cells_cache: dict = {}
_child_cache: dict = {}


def _morton(ijk, depth):
    k = torch.zeros(ijk.shape[0], dtype=torch.int64, device=ijk.device)
    for b in range(depth):
        for a in range(3):
            k |= ((ijk[:, a] >> b) & 1) << (3 * b + 2 - a)
    return k


def _cells(case):
    """(n, 3) int64 finest-level coordinates of the leaves, in Morton order."""
    key = (case["scene"], case.get("geom", 0), case["depth"])
    if key in _cells_cache:
        return _cells_cache[key]
    depth = case["depth"]
    n = 1 << depth
    h = 2.0 / n
    x = (torch.arange(n, dtype=torch.float64, device=DEV) + 0.5) * h - 1.0
    out = []
    if case["scene"] == "spheres":
        rng = np.random.default_rng(0)
        mu, r = rng.uniform(-0.6, 0.6, (3, 3)), rng.uniform(0.2, 0.4, 3)
        sdf = torch.full((n, n, n), math.inf, dtype=torch.float64, device=DEV)
        for m, q in zip(mu, r):
            d2 = ((x - m[0]) ** 2)[:, None, None] + ((x - m[1]) ** 2)[None, :, None] + ((x - m[2]) ** 2)[None, None, :]
            sdf = torch.minimum(sdf, d2.sqrt() - q)
        out.append(torch.nonzero(sdf.abs() <= h))
    else:
        rng = np.random.default_rng(case["geom"])
        mu = torch.from_numpy(rng.uniform(-0.62, 0.62, (20, 3))).to(DEV)
        s = torch.from_numpy(rng.uniform(0.13, 0.24, 20)).to(DEV)
        amp = torch.from_numpy(rng.uniform(0.7, 1.3, 20)).to(DEV)
        d = x[None, None, :] - mu[:, :, None]                       # blob, axis, index
        g = torch.exp(-d * d / (2 * s[:, None, None] ** 2))
        g[:, 0] *= amp[:, None]
        q = -d / s[:, None, None] ** 2
        for i0 in range(0, n, 32):                                  # slabs along x
            gx, qx = g[:, 0, i0:i0 + 32], q[:, 0, i0:i0 + 32]
            yz = (g[:, 1, :, None] * g[:, 2, None, :]).reshape(20, -1)
            yqz = ((g[:, 1] * q[:, 1])[:, :, None] * g[:, 2, None, :]).reshape(20, -1)
            yzq = (g[:, 1, :, None] * (g[:, 2] * q[:, 2])[:, None, :]).reshape(20, -1)
            f = gx.T @ yz
            gn = ((((gx * qx).T @ yz) ** 2) + (gx.T @ yqz) ** 2 + (gx.T @ yzq) ** 2).sqrt()
            ok = ((f - 0.3).abs() <= 2.0 * h * gn).reshape(-1, n, n)
            c = torch.nonzero(ok)
            c[:, 0] += i0
            out.append(c)
    ijk = torch.cat(out)
    ijk = ijk[torch.argsort(_morton(ijk, depth))].contiguous()
    if len(_cells_cache) >= 8:
        _cells_cache.pop(next(iter(_cells_cache)))
    _cells_cache[key] = ijk
    return ijk


def _child(case):
    """The octree's child array over _cells(case), which it numbers in their order."""
    key = (case["scene"], case.get("geom", 0), case["depth"])
    if key not in _child_cache:
        ijk = _cells(case).cpu().numpy()
        cells = np.concatenate([np.full((len(ijk), 1), case["depth"]), ijk], 1).astype(np.int32)
        child, perm = po.build_host(case["depth"], case["degree"], cells)
        assert np.array_equal(perm, np.arange(len(ijk)))
        if len(_child_cache) >= 8:
            _child_cache.pop(next(iter(_child_cache)))
        _child_cache[key] = child
    return _child_cache[key]


# --------------------------------------------------------------- drawn inputs

def _gen(seed, salt):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 1000 + salt)


def _leaves(case, seed, salt=0):
    """Leaf values on the GPU: sigma (n,), records (n, stride), and lobes or a codebook."""
    n, K = _cells(case).shape[0], (case["degree"] + 1) ** 2
    g = _gen(seed, salt)
    sigma = torch.exp(2.0 + torch.randn(n, generator=g, device=DEV))
    lobes = codebook = None
    if case["leaf"] == "codebook":
        M = 16384
        codebook = (0.5 * torch.randn((K, M, 4), generator=g, device=DEV)).half()
        codebook[:, :, 3] = 0
        rec = torch.zeros((n, (K + 3) // 4 * 4), dtype=torch.int16, device=DEV)
        rec[:, :K] = torch.randint(0, M, (n, K), generator=g, device=DEV).to(torch.int16)
        return sigma.half(), rec, None, codebook
    rec = torch.zeros((n, (3 * K + 3) // 4 * 4), device=DEV)
    rec[:, :3 * K] = 0.5 * torch.randn((n, 3 * K), generator=g, device=DEV)
    if case["leaf"] == "sg":
        p = torch.randn((K, 3), generator=g, device=DEV)
        p = p / p.norm(dim=1, keepdim=True)
        lobes = torch.cat([p, 2.0 + 10.0 * torch.rand((K, 1), generator=g, device=DEV)], 1).contiguous()
    if case["leaf"] == "f16":
        sigma, rec = sigma.half(), rec.half()
    return sigma, rec, lobes, codebook


def _pose(seed, salt):
    rng = np.random.default_rng([int(seed), salt])
    z, phi = rng.uniform(0.0, 1.0), rng.uniform(0.0, 2 * math.pi)
    eye = 4.0 * np.array([math.sqrt(1 - z * z) * math.cos(phi), math.sqrt(1 - z * z) * math.sin(phi), z])
    f = -eye / np.linalg.norm(eye)
    r = np.cross(f, [0.0, 0.0, 1.0])
    r /= np.linalg.norm(r)
    return np.stack([r, np.cross(r, f), -f, eye], 1).astype(np.float32)


def _camera(c2w, W, H):
    f = 0.5 * W / math.tan(math.radians(20.0))
    return po.Camera(c2w, W, H, f, f, 0.5 * W, 0.5 * H)


def _pixel_rays(c2w, W, H):
    """Float64 pixel-centre rays (H*W, 3) of a camera given in float32."""
    f = float(np.float32(0.5 * W / math.tan(math.radians(20.0))))
    M = torch.from_numpy(np.asarray(c2w, np.float64)).to(DEV)
    v, u = torch.meshgrid(torch.arange(H, dtype=torch.float64, device=DEV),
                          torch.arange(W, dtype=torch.float64, device=DEV), indexing="ij")
    d = torch.stack([(u + 0.5 - 0.5 * W) / f, -(v + 0.5 - 0.5 * H) / f, torch.full_like(u, -1.0)], -1).reshape(-1, 3)
    return M[:, 3].expand(d.shape[0], 3).contiguous(), (d @ M[:, :3].T).contiguous()


def _free_rays(n, seed, salt):
    """Rays from a sphere of radius 3 towards points of the box, some missing it."""
    g = _gen(seed, salt)
    v = torch.randn((n, 3), generator=g, device=DEV)
    o = 3.0 * v / v.norm(dim=1, keepdim=True)
    t = 2.4 * torch.rand((n, 3), generator=g, device=DEV) - 1.2
    d = (t - o) * (0.5 + 1.5 * torch.rand((n, 1), generator=g, device=DEV))
    return o.contiguous(), d.contiguous()


def _train_data(case, seed):
    """All pixels of six 400x400 training views: rays and target colours."""
    o, d = [], []
    for k in range(6):
        a, b = _pixel_rays(_pose(seed, 100 + k), 400, 400)
        o.append(a.float())
        d.append((b / b.norm(dim=1, keepdim=True)).float())
    o, d = torch.cat(o), torch.cat(d)
    t = 0.5 + 0.4 * torch.sin(9.0 * d + torch.tensor([0.0, 1.0, 2.0], device=DEV))
    t = t + 0.05 * torch.randn(t.shape, generator=_gen(seed, 9), device=DEV)
    return o, d, t.float().contiguous()


CLIP = (0.6, 0.0, 0.8, 0.1)
LR = 1e6


def _job_case(case, j):
    """Every third request of a batch is of the other resident scene."""
    return dict(case, geom=12, depth=7) if j % 3 == 2 else case


# ----------------------------------------------------------------- one pass

def _tree(case, values):
    sigma, rec, lobes, codebook = values
    child = torch.from_numpy(_child(case)).to(DEV)
    return po.Tree(case["depth"], case["degree"], child, sigma, rec, lobes=lobes, codebook=codebook)


def prepare(case, seed):
    tree = _tree(case, _leaves(case, seed))
    s = dict(case=case, tree=tree)
    kind = case["kind"]
    if kind in ("view", "viewer", "filter"):
        s["cam"] = _camera(_pose(seed, 1), case["W"], case["H"])
    if kind == "filter":
        s["weight"] = torch.zeros(tree.n_leaves, device=DEV)
        s["alpha"] = torch.empty((case["H"], case["W"]), device=DEV)
    if kind in ("rays", "grad"):
        s["o"], s["d"] = _free_rays(case["n"], seed, 2)
    if kind == "grad":
        s["g"] = torch.randn((case["n"], 3), generator=_gen(seed, 3), device=DEV)
        tree.sigma.requires_grad_()
        tree.sh.requires_grad_()
    if kind == "train":
        s["fit"] = Trainer(tree, *_train_data(case, seed), lr_sigma=LR, lr_sh=LR, batch=case["n"], seed=seed)
    if kind == "batch":
        other = _tree(_job_case(case, 2), _leaves(_job_case(case, 2), seed, 5))
        s["other"] = other
        s["jobs"] = [po.Job(other if j % 3 == 2 else tree, _camera(_pose(seed, 20 + j), case["W"], case["H"]),
                            torch.empty((case["H"], case["W"], 3), device=DEV), one_pass=True)
                     for j in range(case["jobs"])]
    return s


def run(s):
    case, tree = s["case"], s["tree"]
    kind = case["kind"]
    if kind == "view":
        return po.render_camera(tree, s["cam"])
    if kind == "viewer":
        return po.render_camera(tree, s["cam"], aux=True, sh_off=case["sh_off"], clip=CLIP if case["clip"] else None)
    if kind == "rays":
        return po.render_rays(tree, s["o"], s["d"])
    if kind == "grad":
        rgb = po.render_rays_differentiable(tree, s["o"], s["d"])
        gs, gh = torch.autograd.grad(rgb, (tree.sigma, tree.sh), s["g"])
        return rgb.detach(), gs, gh
    if kind == "train":
        loss = s["fit"].step()
        return loss, tree.sigma, tree.sh
    if kind == "filter":
        s["weight"].zero_()
        leaf_weights(tree, [s["cam"]], weight=s["weight"], alpha_out=[s["alpha"]])
        return s["weight"], s["alpha"]
    po.render_batch(s["jobs"])
    return [j.out for j in s["jobs"]]


# ------------------------------------------------------------- necessary work

def work(case):
    """One pass: about 8 data samples a ray through the blob band whatever the
    depth (3 through the spheres' shells); each record that is met is read
    once, each output written once."""
    K = (case["degree"] + 1) ** 2
    kind = case["kind"]
    rays = case["n"] if "n" in case else case["W"] * case["H"] * case.get("jobs", 1)
    S = rays * (3.0 if case["scene"] == "spheres" else 8.0)
    leaves = 2090.0 if case["scene"] == "spheres" else 10.9 * 4.0 ** case["depth"]
    met = leaves * (1.0 - math.exp(-S / leaves))
    rec = {"f32": 4 * (1 + 3 * K), "sg": 4 * (1 + 3 * K), "f16": 2 * (1 + 3 * K), "codebook": 2 * (1 + K)}[case["leaf"]]
    flops = S * (6.0 * K + 25.0)
    by = met * rec + rays * 12.0
    if kind == "viewer":
        by += rays * 16.0
    if kind in ("rays", "grad", "train"):
        by += rays * 24.0
    if kind == "grad":
        by += leaves * rec + rays * 12.0
        flops *= 2.5
    if kind == "train":                 # parameters read and written, gradients of the met ones
        by += 2.0 * leaves * rec + met * rec + rays * 12.0
        flops = flops * 2.5 + 2.0 * leaves * (1 + 3 * K)
    if kind == "filter":
        by = met * 4.0 + leaves * 4.0 + rays * 4.0
        flops = S * 8.0
    return {"bytes": by, "flops": flops}


# ---------------------------------------------------- float64 results in torch

def _grids(case):
    """Dense finest-level grids: leaf number (-1: empty), and for every empty
    cell the number of levels up to the largest empty octree cube holding it."""
    D = case["depth"]
    n = 1 << D
    ijk = _cells(case)
    leaf = torch.full((n, n, n), -1, dtype=torch.int32, device=DEV)
    leaf[ijk[:, 0], ijk[:, 1], ijk[:, 2]] = torch.arange(ijk.shape[0], dtype=torch.int32, device=DEV)
    up = torch.zeros((n, n, n), dtype=torch.uint8, device=DEV)
    occ = leaf >= 0
    for k in range(1, D):               # cubes of 2^k cells; the root is never a cell
        m = n >> k
        occ = occ.view(m, 2, m, 2, m, 2).amax((1, 3, 5)) if occ.dtype != torch.bool else \
            occ.view(m, 2, m, 2, m, 2).any(5).any(3).any(1)
        free = ~occ
        up.view(m, 1 << k, m, 1 << k, m, 1 << k).masked_fill_(free[:, None, :, None, :, None], k)
    return leaf.view(-1), up.view(-1)


def _sh64(d, K):
    x, y, z = d.unbind(1)
    one = torch.ones_like(x)
    pi = math.pi
    Y = [0.5 * math.sqrt(1 / pi) * one]
    if K > 1:
        c = math.sqrt(3 / (4 * pi))
        Y += [c * y, c * z, c * x]
    if K > 4:
        Y += [0.5 * math.sqrt(15 / pi) * x * y, 0.5 * math.sqrt(15 / pi) * y * z,
              0.25 * math.sqrt(5 / pi) * (3 * z * z - 1), 0.5 * math.sqrt(15 / pi) * x * z,
              0.25 * math.sqrt(15 / pi) * (x * x - y * y)]
    if K > 9:
        a, b = 0.25 * math.sqrt(35 / (2 * pi)), 0.25 * math.sqrt(21 / (2 * pi))
        Y += [a * y * (3 * x * x - y * y), 0.5 * math.sqrt(105 / pi) * x * y * z, b * y * (5 * z * z - 1),
              0.25 * math.sqrt(7 / pi) * z * (5 * z * z - 3), b * x * (5 * z * z - 1),
              0.25 * math.sqrt(105 / pi) * z * (x * x - y * y), a * x * (x * x - 3 * y * y)]
    return torch.stack(Y, 1)


class _Scene64:
    """Leaf values in float64 and the colour basis of a case."""

    def __init__(self, case, values):
        self.case, self.K = case, (case["degree"] + 1) ** 2
        self.sigma, self.rec, self.lobes, self.codebook = values

    def basis(self, d):
        if self.lobes is None:
            return _sh64(d, self.K)
        p = self.lobes.double()
        ax = p[:, :3] / p[:, :3].norm(dim=1, keepdim=True)
        return torch.exp(p[:, 3] * (d @ ax.T - 1.0))

    def coef(self, leaf):
        if self.codebook is not None:
            pos = self.rec[leaf, :self.K].long()
            return torch.stack([self.codebook[k, pos[:, k], :3] for k in range(self.K)], 2).double()
        return self.rec[leaf, :3 * self.K].double().view(-1, 3, self.K)


def _walk(case, o, d, visit, clip=None):
    """Front-to-back octree walk of float64 rays.  visit(rays, leaf, t0, t1)
    gets the data segments of one step (distances along the unit direction)
    and returns which of these rays stop.  Returns the cells stepped per ray."""
    leaf_grid, up_grid = _grids(case)
    D = case["depth"]
    N = 1 << D
    n = o.shape[0]
    ln = d.norm(dim=1)
    og, dg = (o + 1.0) * (N / 2.0), d * (N / 2.0)
    dg = torch.where(dg == 0, torch.full_like(dg, 1e-300), dg)
    inv = 1.0 / dg
    ta, tb = (0.0 - og) * inv, (N - og) * inv
    s0 = torch.minimum(ta, tb).amax(1).clamp_min(0.0)
    s1 = torch.maximum(ta, tb).amin(1)
    hi = torch.full_like(s0, 1e300)
    if clip is not None:
        nv = torch.tensor([float(np.float32(v)) for v in clip], dtype=torch.float64, device=DEV)
        p0, pd = o @ nv[:3] + nv[3], d @ nv[:3]
        t = -p0 / pd
        s0 = torch.where(pd > 0, torch.maximum(s0, t), s0)
        hi = torch.where(pd < 0, t, hi)
        s1 = torch.minimum(s1, hi)
    steps = torch.zeros(n, dtype=torch.float64, device=DEV)
    idx = torch.nonzero(s1 > s0)[:, 0]
    og, dg, inv, s, ln, hi = og[idx], dg[idx], inv[idx], s0[idx], ln[idx], hi[idx]
    c = torch.floor(og + s[:, None] * dg).clamp(0, N - 1).long()
    while idx.numel():
        lin = (c[:, 0] * N + c[:, 1]) * N + c[:, 2]
        leaf, up = leaf_grid[lin].long(), up_grid[lin].long()
        size = torch.where(leaf >= 0, torch.ones_like(up), torch.ones_like(up) << up)[:, None]
        lo = c // size * size
        pos = dg > 0
        sk = (torch.where(pos, lo + size, lo).double() - og) * inv
        se = torch.minimum(torch.maximum(sk.amin(1), s), hi)
        steps[idx] += 1
        q = torch.floor(og + se[:, None] * dg).long()
        q = torch.minimum(torch.maximum(q, lo), lo + size - 1)
        q = torch.where(pos, torch.maximum(q, c), torch.minimum(q, c))
        cross = sk <= se[:, None]
        c = torch.where(cross, torch.where(pos, lo + size, lo - 1), q)
        go = ((c >= 0) & (c < N)).all(1) & (se < hi)
        data = torch.nonzero((leaf >= 0) & (se > s))[:, 0]
        if data.numel():
            stop = visit(idx[data], leaf[data], s[data] * ln[data], se[data] * ln[data])
            go[data[stop]] = False
        s = se
        keep = torch.nonzero(go)[:, 0]
        if keep.numel() < idx.numel():
            idx, c, og, dg, inv, s, ln, hi = (v[keep] for v in (idx, c, og, dg, inv, s, ln, hi))
    return steps


def _render64(case, scene, o, d, sh_off=0, clip=None, stop_T=STOP_T):
    """Colours on white, and the aux columns (T, samples, cells, depth)."""
    n = o.shape[0]
    C = torch.zeros((n, 3), dtype=torch.float64, device=DEV)
    T = torch.ones(n, dtype=torch.float64, device=DEV)
    ns, dep = torch.zeros_like(T), torch.zeros_like(T)
    unit = d / d.norm(dim=1, keepdim=True)
    st = float(np.float32(stop_T))
    keep = torch.tensor([0.0 if (sh_off >> k) & 1 else 1.0 for k in range(scene.K)], dtype=torch.float64, device=DEV)

    def visit(r, leaf, t0, t1):
        sg = scene.sigma[leaf].double().clamp_min(0.0)
        tau = sg * (t1 - t0)
        ex = torch.exp(-tau)
        al = -torch.expm1(-tau)
        Tr = T[r]
        col = torch.sigmoid((scene.coef(leaf) * (scene.basis(unit[r]) * keep)[:, None, :]).sum(2))
        C[r] += (Tr * al)[:, None] * col
        ns[r] += 1
        dep[r] += Tr * (t0 * al + torch.where(sg > 0, al / sg.clamp_min(1e-300) - (t1 - t0) * ex, 0.0))
        T[r] = Tr * ex
        return (T[r] < st) & (sg > 0)

    steps = _walk(case, o, d, visit, clip)
    return C + T[:, None], torch.stack([T, ns, steps, dep], 1)


def _grad64(case, scene, o, d, C, g, stop_T=STOP_T):
    """Gradients of sum(g * colour) for the raw densities and the records."""
    n = o.shape[0]
    P = torch.zeros((n, 3), dtype=torch.float64, device=DEV)
    T = torch.ones(n, dtype=torch.float64, device=DEV)
    gs = torch.zeros(scene.sigma.shape, dtype=torch.float64, device=DEV)
    gh = torch.zeros(scene.rec.shape, dtype=torch.float64, device=DEV)
    unit = d / d.norm(dim=1, keepdim=True)
    st = float(np.float32(stop_T))

    def visit(r, leaf, t0, t1):
        sg = scene.sigma[leaf].double()
        on = sg > 0
        tau = sg.clamp_min(0.0) * (t1 - t0)
        Tn = T[r] * torch.exp(-tau)
        w = T[r] * -torch.expm1(-tau)
        Y = scene.basis(unit[r])
        col = torch.sigmoid((scene.coef(leaf) * Y[:, None, :]).sum(2))
        P[r] += w[:, None] * col
        G = (t1 - t0) * (g[r] * (col * Tn[:, None] - (C[r] - P[r]))).sum(1)
        gs.index_add_(0, leaf, torch.where(on, G, 0.0))
        z = g[r] * w[:, None] * col * (1 - col)
        full = torch.zeros((leaf.numel(), gh.shape[1]), dtype=torch.float64, device=DEV)
        full[:, :3 * scene.K] = (z[:, :, None] * Y[:, None, :]).reshape(leaf.numel(), -1)
        gh.index_add_(0, leaf, full)
        T[r] = Tn
        return (Tn < st) & on

    _walk(case, o, d, visit)
    return gs, gh


def _batch_rows(seed, n, n_src):
    """Rows floor(z n_src / 2^64) of the first n SplitMix64 outputs of `seed`."""
    m = (1 << 64) - 1
    with np.errstate(over="ignore"):
        z = np.uint64(seed & m) + np.arange(1, n + 1, dtype=np.uint64) * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z = z ^ (z >> np.uint64(31))
    hi, lo = z >> np.uint64(32), z & np.uint64(0xFFFFFFFF)
    s = np.uint64(n_src)                # n_src < 2^32
    return torch.from_numpy(((hi * s + ((lo * s) >> np.uint64(32))) >> np.uint64(32)).astype(np.int64)).to(DEV)


@torch.no_grad()
def exact(case, seed):
    kind = case["kind"]
    scene = _Scene64(case, _leaves(case, seed))
    if kind in ("view", "viewer"):
        o, d = _pixel_rays(_pose(seed, 1), case["W"], case["H"])
        img, aux = _render64(case, scene, o, d, case.get("sh_off", 0), CLIP if case.get("clip") else None)
        img = img.view(case["H"], case["W"], 3)
        return img if kind == "view" else (img, aux.view(case["H"], case["W"], 4))
    if kind == "rays":
        o, d = _free_rays(case["n"], seed, 2)
        return _render64(case, scene, o.double(), d.double())[0]
    if kind == "grad":
        o, d = (v.double() for v in _free_rays(case["n"], seed, 2))
        g = torch.randn((case["n"], 3), generator=_gen(seed, 3), device=DEV).double()
        C = _render64(case, scene, o, d)[0]
        return (C, *_grad64(case, scene, o, d, C, g))
    if kind == "train":
        o, d, t = _train_data(case, seed)
        rows = _batch_rows(int(seed), case["n"], o.shape[0])
        o, d, t = o[rows].double(), d[rows].double(), t[rows].double()
        C = _render64(case, scene, o, d)[0]
        e = C - t
        gs, gh = _grad64(case, scene, o, d, C, 2.0 * e / (3 * case["n"]))
        return (e * e).sum().view(1) / (3 * case["n"]), scene.sigma.double() - LR * gs, scene.rec.double() - LR * gh
    if kind == "filter":
        o, d = _pixel_rays(_pose(seed, 1), case["W"], case["H"])
        T = torch.ones(o.shape[0], dtype=torch.float64, device=DEV)
        w = torch.zeros(scene.sigma.shape, dtype=torch.float64, device=DEV)
        st = float(np.float32(STOP_T))

        def visit(r, leaf, t0, t1):
            tau = scene.sigma[leaf].double().clamp_min(0.0) * (t1 - t0)
            w.scatter_reduce_(0, leaf, -torch.expm1(-tau), "amax")
            T[r] *= torch.exp(-tau)
            return (T[r] < st) & (tau > 0)

        _walk(case, o, d, visit)
        return w, (1.0 - T).view(case["H"], case["W"])
    other = _Scene64(_job_case(case, 2), _leaves(_job_case(case, 2), seed, 5))
    out = []
    for j in range(case["jobs"]):
        o, d = _pixel_rays(_pose(seed, 20 + j), case["W"], case["H"])
        jc = _job_case(case, j)
        out.append(_render64(jc, other if j % 3 == 2 else scene, o, d)[0].view(case["H"], case["W"], 3))
    return out
