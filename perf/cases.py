"""Timed cases of the select / recolour / render / refit path, through the package's
public entry points, over the range of sizes its users have: editing frames from a
4,096-Gaussian preview to three million Gaussians, the batched viewer, the multi-view
gradient, the SH refit in both of its forms, the loss, the point-cloud filter, the whole
selection chain, and baking an edit into a copy of a scene.

`listed()` names the cases, `draw(rng)` gives another one of the same ranges,
`prepare(case, seed)` makes what a program has in hand before the call, `run(state)` is
one pass, `work(case)` the bytes and operations it cannot do without, `exact(case, seed)`
its outputs in 64 bits by plain torch.
"""
import math
import random

import numpy as np
import torch

import paper_2511_18441_amd as R

DEV = "cuda"
Y00 = 0.28209479177387814
DTYPE = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
SIZE = {"f32": 4, "f16": 2, "bf16": 2}
LAMBDA = 0.2            # weight of the SSIM term of the refit's loss
LR, BETA1, BETA2, EPS, STEP = 2e-3, 0.9, 0.999, 1e-15, 100


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # a preview thumbnail of a small asset: latency and launches are all of it
        dict(name="frame preview 4k 128", kind="frame", n=4096, deg=0, storage="f32", w=128, h=128, tile_w=16, tile_h=16,
             ppt=1, graph=False, edit="fused", select=True),
        # an editor's interactive view while the brush moves: select and tint in every frame
        dict(name="frame editor 200k 800", kind="frame", n=200_000, deg=3, storage="f32", w=800, h=800, tile_w=16,
             tile_h=16, ppt=1, graph=False, edit="fused", select=True),
        # the viewer's frame: recolour the selected coefficients, render the edited scene
        dict(name="frame viewer 1M 1080p f32", kind="frame", n=1_000_000, deg=3, storage="f32", w=1920, h=1080,
             tile_w=32, tile_h=32, ppt=1, graph=True, edit="recolor", select=False),
        # the same on a compressed scene of odd size at a laptop's resolution
        dict(name="frame odd 777k 1366 bf16", kind="frame", n=777_777, deg=2, storage="bf16", w=1366, h=768, tile_w=32,
             tile_h=32, ppt=1, graph=True, edit="recolor", select=False),
        # a server drawing 8 scenes of uneven size from 4 cameras each in one batch
        dict(name="batch 8 scenes x 4 f16", kind="batch",
             sizes="100000,250000,500000,1000000,1000000,1500000,2000000,3000000",
             res="256x256,800x800,1280x720,1920x1080", deg=3, storage="f16", tile_w=32, tile_h=32, ppt=1),
        # gradient of a two-view loss in opacity, DC colour and recolour matrix
        dict(name="gradient 1M 720p x2", kind="diff", n=1_000_000, deg=3, storage="f32", w=1280, h=720, views=2,
             tile_w=32, tile_h=16, ppt=1),
        # one step of the background optimiser, loss and Adam step fused
        dict(name="refit fused 1M 720p", kind="refit", n=1_000_000, deg=3, w=1280, h=720, tile_w=32, tile_h=16, ppt=1,
             fused=True, graph=True),
        # one step on a small asset at a ragged size, the optimiser's pieces called one by one
        dict(name="refit pieces 20k 333x217", kind="refit", n=20_011, deg=3, w=333, h=217, tile_w=16, tile_h=16, ppt=1,
             fused=False, graph=False),
        # the loss alone on a full frame
        dict(name="loss 1080p", kind="loss", w=1920, h=1080),
        # cleaning an unprojected selection
        dict(name="cloud filter 314k k16", kind="cloud", n=314_218, k=16),
        # the selection chain: rough depth, brush to cloud, clean, mask in another view, tint
        dict(name="selection chain 1M 1080p", kind="select", n=1_000_000, deg=3, storage="f32", w=1920, h=1080,
             brush=0.35, tile_w=32, tile_h=32, ppt=1),
        # opening a scene and baking an edit into a whole copy of it
        dict(name="bake 3M f16", kind="bake", n=3_000_000, deg=3, storage="f16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["frame", "frame", "frame", "batch", "diff", "refit", "refit", "loss", "cloud", "select", "bake"])
    w = _log(rng, 96, 1920)
    h = max(64, min(1080, int(w * rng.uniform(0.5, 1.0))))
    tile_w, tile_h = rng.choice([(16, 16), (32, 16), (32, 32)])
    shape = dict(w=w, h=h, tile_w=tile_w, tile_h=tile_h, ppt=1)
    if kind == "frame":
        edit = rng.choice(["none", "fused", "recolor"])
        return dict(kind=kind, n=_log(rng, 4096, 1_500_000), deg=rng.choice([0, 1, 2, 3, 3, 3]),
                    storage=rng.choice(["f32", "f32", "f16", "bf16"]), graph=rng.random() < 0.5, edit=edit,
                    select=edit == "fused" and rng.random() < 0.5, **shape)
    if kind == "batch":
        sizes = ",".join(str(_log(rng, 50_000, 1_000_000)) for _ in range(rng.randint(1, 4)))
        res = ",".join("%dx%d" % (_log(rng, 200, 1280), _log(rng, 160, 720)) for _ in range(rng.randint(2, 4)))
        return dict(kind=kind, sizes=sizes, res=res, deg=3, storage=rng.choice(["f16", "f32", "bf16"]), tile_w=32,
                    tile_h=32, ppt=rng.choice([1, 2]))
    if kind == "diff":
        return dict(kind=kind, n=_log(rng, 4096, 1_000_000), deg=rng.choice([0, 1, 3]),
                    storage=rng.choice(["f32", "f16"]), views=rng.randint(1, 3), **dict(shape, tile_w=rng.choice([16, 32]),
                                                                                        tile_h=16))
    if kind == "refit":
        return dict(kind=kind, n=_log(rng, 4096, 1_000_000), deg=rng.choice([1, 2, 3, 3]), fused=rng.random() < 0.6,
                    graph=rng.random() < 0.6, **dict(shape, tile_w=rng.choice([16, 32]), tile_h=16))
    if kind == "loss":
        return dict(kind=kind, w=w, h=h)
    if kind == "cloud":
        return dict(kind=kind, n=_log(rng, 2000, 400_000), k=rng.choice([8, 16, 16, 32]))
    if kind == "select":
        return dict(kind=kind, n=_log(rng, 50_000, 1_000_000), deg=rng.choice([1, 3]), storage=rng.choice(["f32", "f16"]),
                    brush=round(rng.uniform(0.1, 0.4), 3), **dict(shape, w=max(w, 320), h=max(h, 240)))
    return dict(kind="bake", n=_log(rng, 20_000, 2_500_000), deg=rng.choice([0, 1, 2, 3]),
                storage=rng.choice(["f32", "f16", "bf16"]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
class Camera:
    """A pinhole camera on an orbit around the origin, looking at it (60 degrees wide)."""

    def __init__(self, width, height, az, el, radius=4.0):
        C = radius * np.array([math.cos(el) * math.sin(az), math.sin(el), math.cos(el) * math.cos(az)])
        zc = -C / np.linalg.norm(C)
        xc = np.cross(zc, np.array([0.0, 1.0, 0.0]))
        xc /= np.linalg.norm(xc)
        self.R = np.stack([xc, np.cross(zc, xc), zc]).astype(np.float32)
        self.t = (-(self.R.astype(np.float64) @ C)).astype(np.float32)
        self.width, self.height = width, height
        self.fx = self.fy = float(np.float32((width / 2.0) / math.tan(math.radians(30.0))))
        self.cx, self.cy, self.znear = width / 2.0, height / 2.0, float(np.float32(0.2))


class Select:
    """A brush disk on the screen and a ball around a reference colour."""

    def __init__(self, rng, width, height, radius):
        self.cx, self.cy, self.radius = width / 2.0, height / 2.0, float(np.float32(radius * min(width, height)))
        self.ref = np.float32([rng.uniform(0.2, 0.8) for _ in range(3)])
        self.color_radius = float(np.float32(0.3))


def _cameras(seed, sizes):
    rng = random.Random(seed * 7919 + 1)
    return [Camera(w, h, rng.uniform(0, 2 * math.pi), math.radians(rng.uniform(10, 35))) for w, h in sizes]


def _select(seed, w, h):
    return Select(random.Random(seed * 7919 + 2), w, h, 0.12)


def _gen(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 64 + salt)
    return g


def _arrays(seed, n, deg, storage, salt=0):
    """Planes of a splat scene: 64 rotated anisotropic clusters and a ground plane (8 round
    clusters of larger splats below 16,384 Gaussians)."""
    g = _gen(seed, salt)

    def rand(*s):
        return torch.rand(*s, generator=g, device=DEV)

    def randn(*s):
        return torch.randn(*s, generator=g, device=DEV)
    quats = randn(4, n)
    quats /= quats.norm(dim=0, keepdim=True)
    if n < 16_384:
        centres = rand(8, 3) * 2 - 1
        member = torch.randint(0, 8, (n,), generator=g, device=DEV)
        means = (centres[member] + 0.2 * randn(n, 3)).T.contiguous()
        log_scales = -3.5 + 0.5 * randn(3, n)
    else:
        nc = int(round(0.8 * n))
        centres, sds = rand(64, 3) * 3 - 1.5, rand(64, 3) * 0.35 + 0.05
        rots = torch.linalg.qr(randn(64, 3, 3).double())[0].float()
        member = torch.randint(0, 64, (nc,), generator=g, device=DEV)
        local = randn(nc, 3) * sds[member]
        cluster = centres[member] + (rots[member] * local[:, None, :]).sum(-1)
        ground = rand(n - nc, 3) * 4 - 2
        ground[:, 1] = -1 + 0.02 * randn(n - nc)
        means = torch.cat([cluster, ground]).T.contiguous()
        log_scales = (-4.5 + 0.6 * randn(3, n)).clamp(-8, -1)
    opacity = torch.sigmoid(1.5 * randn(n)).to(DTYPE[storage])
    sh = 0.05 * randn(3 * (deg + 1) ** 2, n)
    sh[:3] = (rand(3, n) - 0.5) / Y00
    return dict(means=means, log_scales=log_scales, quats=quats, opacity=opacity, sh=sh.to(DTYPE[storage]))


class Scene(R.DeviceScene):
    """A DeviceScene whose planes were made on the GPU."""

    def __init__(self, arrays, deg, storage):
        self.__dict__.update(arrays)
        self.n = self.stride = int(arrays["means"].shape[1])
        self.sh_degree, self.storage = deg, storage
        self.cov3d = torch.empty((6, self.n), device=DEV)
        R.recogs_prepare_covariance(self.log_scales.data_ptr(), self.quats.data_ptr(), self.cov3d.data_ptr(), self.n, self.n)


def _edit(seed):
    rng = np.random.default_rng(seed + 17)
    M = (np.eye(3) + 0.2 * rng.standard_normal((3, 3))).astype(np.float32)
    b = rng.uniform(-0.1, 0.1, 3).astype(np.float32)
    return torch.from_numpy(M.reshape(9)).to(DEV), torch.from_numpy(b).to(DEV)


def _picture(seed, h, w, salt):
    """A smooth picture with fine grain, values in [0, 1]."""
    g = _gen(seed, salt)
    y = torch.linspace(0, 1, h, device=DEV)[:, None, None]
    x = torch.linspace(0, 1, w, device=DEV)[None, :, None]
    p = torch.rand(6, 3, generator=g, device=DEV)
    img = 0.45 + 0.2 * torch.sin(6.3 * (2 * x + p[0]) + 4 * y) + 0.15 * torch.cos(6.3 * (5 * y + p[1]) - 9 * p[2] * x)
    img = img + 0.1 * torch.sin(40 * p[3] * x + 55 * p[4] * y) + 0.03 * torch.randn(h, w, 3, generator=g, device=DEV)
    return img.clamp(0, 1).contiguous()


def _cloud(seed, n):
    """n world points of a brush selection: the pixels of a disk, 70% sampled, at the depths
    of overlapping blobs in front of a wall, with a few flying pixels."""
    g = _gen(seed, 5)
    r = math.sqrt(n / 0.7 / math.pi) + 2.0
    side = int(2 * r) + 3
    yy, xx = torch.meshgrid(torch.arange(side, device=DEV) - side / 2, torch.arange(side, device=DEV) - side / 2, indexing="ij")
    disk = torch.nonzero((xx ** 2 + yy ** 2 <= r * r).reshape(-1)).squeeze(1)
    pick = disk[torch.randperm(disk.numel(), generator=g, device=DEV)[:n]].sort().values
    x, y = xx.reshape(-1)[pick] / r, yy.reshape(-1)[pick] / r
    d = 5.0 + 0.3 * x
    c = torch.rand(24, 4, generator=g, device=DEV)
    for k in range(24):
        q = ((x - 2 * c[k, 0] + 1) ** 2 + (y - 2 * c[k, 1] + 1) ** 2) / (0.15 + 0.4 * c[k, 2]) ** 2
        d = torch.where(q < 1, torch.minimum(d, 3 + 1.8 * c[k, 3] - 0.4 * torch.sqrt((1 - q).clamp(min=0))), d)
    d = d * (1 + 0.004 * torch.randn(n, generator=g, device=DEV))
    fly = torch.rand(n, generator=g, device=DEV) < 0.002
    d = torch.where(fly, d * (0.6 + torch.rand(n, generator=g, device=DEV)), d)
    return torch.stack([0.3 * x * d, 0.3 * y * d, d]).contiguous()


# ---------------------------------------------------------------------------
# prepare / run
# ---------------------------------------------------------------------------
def _tile(c):
    return (c["tile_w"], c["tile_h"])


def _workspace(scene, cam, tile, ppt):
    """A workspace that holds this view's keys (rendered once, as a program's first frame)."""
    ws = R.DeviceWorkspace(scene.n, cam.width, cam.height, tile)
    R.render(scene, cam, ws, tile, ppt)
    return ws


def _zero(*shape, dtype=torch.float32):
    return torch.zeros(shape, dtype=dtype, device=DEV)


def prepare(c, seed):
    kind = c["kind"]
    s = dict(case=c)
    if kind == "loss":
        w, h = c["w"], c["h"]
        nb = R.recogs_dssim_workspace_bytes(w, h)
        return dict(s, image=_picture(seed, h, w, 1), target=_picture(seed, h, w, 2), grad=_zero(h, w, 3), loss=_zero(1),
                    ws=_zero(nb // 4), nb=nb)
    if kind == "cloud":
        return dict(s, points=_cloud(seed, c["n"]), **_filter_buffers(c["n"]))
    if kind == "batch":
        sizes = [int(x) for x in c["sizes"].split(",")]
        res = [tuple(int(v) for v in x.split("x")) for x in c["res"].split(",")]
        scenes = [Scene(_arrays(seed, n, c["deg"], c["storage"], k), c["deg"], c["storage"]) for k, n in enumerate(sizes)]
        cams = _cameras(seed, res * len(sizes))
        M, b = _edit(seed)
        views = []
        for k, cam in enumerate(cams):
            si = k // len(res)
            views.append((si, cam, _mask(seed, scenes[si], cam)[0], M, b))
        return dict(s, batch=R.DeviceBatch(scenes, views, _tile(c), c["ppt"]))
    scene = Scene(_arrays(seed, c["n"], c["deg"], c.get("storage", "f32")), c["deg"], c.get("storage", "f32"))
    s["scene"] = scene
    M, b = _edit(seed)
    s.update(M=M, b=b, mask=_zero(scene.n, dtype=torch.uint8), count=_zero(1, dtype=torch.int32))
    if kind == "bake":
        cam = _cameras(seed, [(1920, 1080)])[0]
        return dict(s, cam=R.camera_struct(cam), sel=R.select_struct(_select(seed, 1920, 1080)), dst=torch.empty_like(scene.sh))
    w, h, tile, ppt = c["w"], c["h"], _tile(c), c["ppt"]
    cams = _cameras(seed, [(w, h)] * c.get("views", 2 if kind == "select" else 1))
    cam = cams[0]
    s.update(cam=cam, image=_zero(h, w, 3))
    if kind == "frame":
        s["ws"] = _workspace(scene, cam, tile, ppt)
        s["sel"] = R.select_struct(_select(seed, w, h))
        s["mask"], s["count"] = _mask(seed, scene, cam)
        if c["edit"] == "recolor":
            s["sh"] = scene.sh.clone()
        return s
    if kind == "diff":
        s["ws"] = [_workspace(scene, k, tile, ppt) for k in cams]
        s["mask"], _ = _mask(seed, scene, cam)
        s.update(cams=cams, images=[_zero(h, w, 3) for _ in cams], targets=[_picture(seed, h, w, 8 + k) for k in range(len(cams))],
                 grad=_zero(h, w, 3), loss=_zero(len(cams)), dop=_zero(scene.n), ddc=_zero(3, scene.n), dM=_zero(9))
        return s
    if kind == "refit":
        g = _gen(seed, 3)
        nb = R.recogs_dssim_workspace_bytes(w, h)
        ncoef = scene.sh.shape[0]
        s.update(ws=_workspace(scene, cam, tile, ppt), target=_picture(seed, h, w, 8), grad=_zero(h, w, 3), loss=_zero(2),
                 sws=_zero(nb // 4), nb=nb, dop=_zero(scene.n), dM=_zero(9), **_moments(g, ncoef, scene.n))
        if not c["fused"]:
            s["dsh"] = _zero(ncoef, scene.n)
        return s
    # select: the second view (its image and rough depth) is in hand
    cam2 = cams[1]
    s.update(cam2=cam2, ws=_workspace(scene, cam, tile, ppt), depth=_zero(h, w), depth2=_zero(h, w), vmask=_zero(h, w, dtype=torch.uint8),
             out=_zero(h, w, 3))
    s["image2"] = R.render(scene, cam2, _workspace(scene, cam2, tile, ppt), tile, ppt, depth=s["depth2"])
    yy, xx = torch.meshgrid(torch.arange(h, device=DEV) + 0.5, torch.arange(w, device=DEV) + 0.5, indexing="ij")
    rad = c["brush"] * min(w, h)
    s["brush"] = (((xx - w / 2) ** 2 + (yy - h / 2) ** 2) <= rad * rad).to(torch.uint8)
    s["keep"] = (torch.rand(h, w, generator=_gen(seed, 4), device=DEV) < 0.7).to(torch.uint8)
    cap = int(s["brush"].sum())
    unb = R.recogs_unproject_workspace_bytes(w, h)
    s.update(cap=cap, cloud=_zero(3, cap), npts=_zero(1, dtype=torch.int32), uws=_zero(unb, dtype=torch.uint8), unb=unb,
             **_filter_buffers(cap))
    return s


def _filter_buffers(n):
    nb = R.recogs_outlier_workspace_bytes(n)
    return dict(dist=_zero(n), kept=_zero(n, dtype=torch.uint8), clean=_zero(3, n), nkept=_zero(1, dtype=torch.int32),
                ows=_zero(nb, dtype=torch.uint8), onb=nb)


def _moments(g, ncoef, n):
    """Adam's moments as a running refit holds them."""
    m = 1e-6 * torch.randn(ncoef, n, generator=g, device=DEV)
    v = (1e-6 * (0.5 + torch.rand(ncoef, n, generator=g, device=DEV))) ** 2
    return dict(m=m, v=v)


def _mask(seed, scene, cam):
    """The Gaussians that the brush selects in this view, and their number."""
    mask, count = _zero(scene.n, dtype=torch.uint8), _zero(1, dtype=torch.int32)
    R.recogs_select(scene.c_struct(), R.camera_struct(cam), R.select_struct(_select(seed, cam.width, cam.height)),
                    mask.data_ptr(), count.data_ptr())
    return mask, count


def run(s):
    c = s["case"]
    return {"frame": _run_frame, "batch": _run_batch, "diff": _run_diff, "refit": _run_refit, "loss": _run_loss,
            "cloud": _run_cloud, "select": _run_select, "bake": _run_bake}[c["kind"]](c, s)


def _run_frame(c, s):
    scene, cam, ws = s["scene"], s["cam"], s["ws"]
    out = {}
    if c["select"]:
        R.recogs_select(scene.c_struct(), R.camera_struct(cam), s["sel"], s["mask"].data_ptr(), s["count"].data_ptr())
        out.update(mask=s["mask"], count=s["count"])
    if c["edit"] == "recolor":
        R.recogs_recolor(scene.c_struct(), s["sh"].data_ptr(), s["mask"].data_ptr(), s["M"].data_ptr(), s["b"].data_ptr(), 0)
        out["sh"] = s["sh"]
        R.render(scene, cam, ws, _tile(c), c["ppt"], image=s["image"], sh=s["sh"], graph_mode=c["graph"])
    elif c["edit"] == "fused":
        R.render(scene, cam, ws, _tile(c), c["ppt"], mask=s["mask"], M=s["M"], b=s["b"], image=s["image"], graph_mode=c["graph"])
    else:
        R.render(scene, cam, ws, _tile(c), c["ppt"], image=s["image"], graph_mode=c["graph"])
    return dict(out, image=s["image"])


def _run_batch(c, s):
    s["batch"].render()
    return s["batch"].images


def _run_diff(c, s):
    scene, tile, ppt, count = s["scene"], _tile(c), c["ppt"], s["grad"].numel()
    opts = R.opts_struct(tile, ppt, mask=s["mask"], M=s["M"], b=s["b"], keep_backward=True)
    for k, cam in enumerate(s["cams"]):
        img = s["images"][k]
        R.render(scene, cam, s["ws"][k], tile, ppt, mask=s["mask"], M=s["M"], b=s["b"], keep_backward=True, image=img, graph_mode=True)
        R.recogs_loss_l2(img.data_ptr(), s["targets"][k].data_ptr(), count, 1.0 / count, s["grad"].data_ptr(),
                         s["loss"].data_ptr() + 4 * k)
        R.recogs_render_backward(scene.c_struct(), R.camera_struct(cam), opts, s["ws"][k].ws, img.data_ptr(), s["grad"].data_ptr(),
                                 s["dop"].data_ptr(), s["ddc"].data_ptr(), s["dM"].data_ptr(), accumulate=int(k > 0))
    return dict(images=s["images"], loss=s["loss"], dop=s["dop"], ddc=s["ddc"], dM=s["dM"])


def _run_refit(c, s):
    scene, cam, tile, ppt = s["scene"], s["cam"], _tile(c), c["ppt"]
    img, tgt, grad, loss, count = s["image"], s["target"], s["grad"], s["loss"], s["grad"].numel()
    opts = R.opts_struct(tile, ppt, keep_backward=True)
    R.render(scene, cam, s["ws"], tile, ppt, keep_backward=True, image=img, graph_mode=c["graph"])
    out = dict(image=img, loss=loss, grad=grad, dop=s["dop"], sh=scene.sh, m=s["m"], v=s["v"])
    sc, cs = scene.c_struct(), R.camera_struct(cam)
    if c["fused"]:
        R.recogs_loss_l1_dssim(img.data_ptr(), tgt.data_ptr(), cam.width, cam.height, (1.0 - LAMBDA) / count, LAMBDA,
                               grad.data_ptr(), 0, loss.data_ptr(), s["sws"].data_ptr(), s["nb"])
        R.recogs_render_backward_sh_adam(sc, cs, opts, s["ws"].ws, img.data_ptr(), grad.data_ptr(), s["dop"].data_ptr(),
                                         s["dM"].data_ptr(), s["m"].data_ptr(), s["v"].data_ptr(), LR, BETA1, BETA2, EPS, STEP)
        return out
    R.recogs_loss_l1(img.data_ptr(), tgt.data_ptr(), count, (1.0 - LAMBDA) / count, grad.data_ptr(), loss.data_ptr())
    R.recogs_loss_dssim(img.data_ptr(), tgt.data_ptr(), cam.width, cam.height, LAMBDA, grad.data_ptr(), 1,
                        loss.data_ptr() + 4, s["sws"].data_ptr(), s["nb"])
    R.recogs_render_backward_sh(sc, cs, opts, s["ws"].ws, img.data_ptr(), grad.data_ptr(), s["dop"].data_ptr(),
                                s["dsh"].data_ptr(), s["dM"].data_ptr())
    R.recogs_adam_step(scene.sh.data_ptr(), s["dsh"].data_ptr(), s["m"].data_ptr(), s["v"].data_ptr(), scene.sh.numel(), LR,
                       BETA1, BETA2, EPS, STEP)
    return dict(out, dsh=s["dsh"])


def _run_loss(c, s):
    count = s["grad"].numel()
    R.recogs_loss_l1_dssim(s["image"].data_ptr(), s["target"].data_ptr(), c["w"], c["h"], (1.0 - LAMBDA) / count, LAMBDA,
                           s["grad"].data_ptr(), 0, s["loss"].data_ptr(), s["ws"].data_ptr(), s["nb"])
    return dict(grad=s["grad"], loss=s["loss"])


def _run_cloud(c, s):
    n = c["n"]
    R.recogs_remove_outliers(s["points"].data_ptr(), n, n, c["k"], 0.007, s["dist"].data_ptr(), s["kept"].data_ptr(),
                             s["clean"].data_ptr(), n, s["nkept"].data_ptr(), s["ows"].data_ptr(), s["onb"])
    return dict(clean=s["clean"], kept=s["kept"], count=s["nkept"], dist=s["dist"])


def _run_select(c, s):
    scene, cam, tile = s["scene"], s["cam"], _tile(c)
    R.render(scene, cam, s["ws"], tile, c["ppt"], image=s["image"], depth=s["depth"], depth_tau=0.5)
    cap, cs = s["cap"], R.camera_struct(cam)
    R.recogs_unproject(cs, s["brush"].data_ptr(), s["keep"].data_ptr(), s["depth"].data_ptr(), s["cloud"].data_ptr(), cap,
                       s["npts"].data_ptr(), s["uws"].data_ptr(), s["unb"])
    n = int(s["npts"].item())
    R.recogs_remove_outliers(s["cloud"].data_ptr(), n, cap, 16, 0.007, s["dist"].data_ptr(), s["kept"].data_ptr(),
                             s["clean"].data_ptr(), cap, s["nkept"].data_ptr(), s["ows"].data_ptr(), s["onb"])
    R.recogs_reproject_mask(R.camera_struct(s["cam2"]), s["clean"].data_ptr(), int(s["nkept"].item()), cap, 2.0,
                            s["depth2"].data_ptr(), 0.01, s["vmask"].data_ptr())
    R.tint(s["image2"], s["vmask"], (1.0, 0.6, 0.5), out=s["out"])
    return dict(image=s["image"], depth=s["depth"], cloud=s["cloud"], points=s["npts"], kept=s["kept"], dist=s["dist"],
                clean=s["clean"], mask=s["vmask"], tinted=s["out"])


def _run_bake(c, s):
    scene = s["scene"]
    R.recogs_prepare_covariance(scene.log_scales.data_ptr(), scene.quats.data_ptr(), scene.cov3d.data_ptr(), scene.n, scene.stride)
    sc = scene.c_struct()
    R.recogs_select(sc, s["cam"], s["sel"], s["mask"].data_ptr(), s["count"].data_ptr())
    R.recogs_recolor(sc, s["dst"].data_ptr(), s["mask"].data_ptr(), s["M"].data_ptr(), s["b"].data_ptr(), 1)
    return dict(cov=scene.cov3d, mask=s["mask"], count=s["count"], sh=s["dst"])


# ---------------------------------------------------------------------------
# work
# ---------------------------------------------------------------------------
def _render_work(n, deg, storage, w, h):
    """Scene in, image out; per Gaussian its projection and colour, per pixel the splats that
    it blends (about 160 in a dense scene before it is opaque, 23 operations each)."""
    ncoef = (deg + 1) ** 2
    evals = min(160.0, 340.0 * n / (w * h)) * w * h
    return n * (36.0 + SIZE[storage] * (1 + 3 * ncoef)) + 12.0 * w * h, n * (200.0 + 6.0 * ncoef) + 23.0 * evals, evals


def work(c):
    kind = c["kind"]
    if kind == "loss":
        px = c["w"] * c["h"]
        return {"bytes": 36.0 * px, "flops": 3.0 * px * (5 * 44 + 3 * 44 + 60)}
    if kind == "cloud":
        return {"bytes": c["n"] * (12.0 + 4 + 1 + 12), "flops": c["n"] * 27.0 * 4 * 8}
    if kind == "bake":
        n, eb, nc = c["n"], SIZE[c["storage"]], 3 * (c["deg"] + 1) ** 2
        return {"bytes": n * (28.0 + 24 + 12 + 2 + 2 * eb * nc), "flops": n * 160.0}
    if kind == "batch":
        sizes = [int(x) for x in c["sizes"].split(",")]
        res = [tuple(int(v) for v in x.split("x")) for x in c["res"].split(",")]
        b = f = 0.0
        for n in sizes:
            b += n * (36.0 + SIZE[c["storage"]] * (1 + 3 * (c["deg"] + 1) ** 2))
            for w, h in res:
                f += _render_work(n, c["deg"], c["storage"], w, h)[1]
                b += 12.0 * w * h + n
        return {"bytes": b, "flops": f}
    n, w, h = c["n"], c["w"], c["h"]
    px = w * h
    b, f, evals = _render_work(n, c["deg"], c.get("storage", "f32"), w, h)
    if kind == "frame":
        return {"bytes": b + n * (1.0 if c["edit"] != "none" else 0.0), "flops": f}
    if kind == "diff":
        # the gradients are read and written once, the scene once a view
        return {"bytes": c["views"] * (b + 24.0 * px + n) + 16.0 * n, "flops": c["views"] * (f + 50.0 * evals)}
    if kind == "refit":
        nc = 3 * (c["deg"] + 1) ** 2
        return {"bytes": b + 24.0 * px + n * (4.0 + 20.0 * nc), "flops": f + 50.0 * evals + 12.0 * n * nc + 1236.0 * px}
    pts = 0.7 * math.pi * (c["brush"] * min(w, h)) ** 2
    return {"bytes": b + 4.0 * px + 2.0 * px + pts * 29.0 + px * (1 + 25.0), "flops": f + pts * 864.0}


# ---------------------------------------------------------------------------
# the same outputs in 64 bits
# ---------------------------------------------------------------------------
def _basis(deg, x, y, z):
    """Real spherical harmonics with the Condon-Shortley phase, l <= deg."""
    p = math.pi
    Y = [torch.full_like(x, 0.5 / math.sqrt(p))]
    if deg >= 1:
        a = math.sqrt(3 / p) / 2
        Y += [-a * y, a * z, -a * x]
    if deg >= 2:
        a, b, c = math.sqrt(15 / p) / 2, math.sqrt(5 / p) / 4, math.sqrt(15 / p) / 4
        Y += [a * x * y, -a * y * z, b * (3 * z * z - 1), -a * x * z, c * (x * x - y * y)]
    if deg >= 3:
        a, b = math.sqrt(35 / (2 * p)) / 4, math.sqrt(105 / p) / 2
        c, d, e = math.sqrt(21 / (2 * p)) / 4, math.sqrt(7 / p) / 4, math.sqrt(105 / p) / 4
        Y += [-a * y * (3 * x * x - y * y), b * x * y * z, -c * y * (5 * z * z - 1), d * z * (5 * z * z - 3),
              -c * x * (5 * z * z - 1), e * z * (x * x - y * y), -a * x * (x * x - 3 * y * y)]
    return torch.stack(Y)


def _cov64(ls, q):
    q = q.double()
    w, x, y, z = q / q.norm(dim=0, keepdim=True)
    rot = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                       2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                       2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]).view(3, 3, -1)
    m = rot * torch.exp(ls.double())[None]
    return [(m[i] * m[j]).sum(0) for i, j in ((0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2))]


def _cam64(cam):
    return torch.from_numpy(cam.R.astype(np.float64)).to(DEV), torch.from_numpy(cam.t.astype(np.float64)).to(DEV)


def _mask64(seed, a, cam):
    rot, t = _cam64(cam)
    m = rot @ a["means"].double() + t[:, None]
    sel = _select(seed, cam.width, cam.height)
    u, v = cam.fx * m[0] / m[2] + cam.cx, cam.fy * m[1] / m[2] + cam.cy
    dc = Y00 * a["sh"][:3].double() + 0.5 - torch.from_numpy(sel.ref.astype(np.float64)).to(DEV)[:, None]
    return (m[2] > cam.znear) & ((u - sel.cx) ** 2 + (v - sel.cy) ** 2 <= sel.radius ** 2) & (dc.square().sum(0) <= sel.color_radius ** 2)


def _recolor64(sh, mask, M, b):
    """The coefficients whose displayed colour is M times the old one plus b, where masked."""
    M, b = M.double().view(3, 3), b.double()
    C = sh.view(-1, 3, sh.shape[1])
    out = (M[None, :, :, None] * C[:, None]).sum(2)
    out[0] += (((M.sum(1) - 1) * 0.5 + b) / Y00)[:, None]
    return torch.where(mask[None, None], out, C).reshape(sh.shape)


class Render64:
    """The image of a scene by its definition, tile by tile, and the gradients of sum(g y)."""

    def __init__(self, a, cam, deg, sh=None, mask=None, M=None, b=None):
        rot, t = _cam64(cam)
        means = a["means"].double()
        self.n, self.cam, W, H = means.shape[1], cam, cam.width, cam.height
        m = rot @ means + t[:, None]
        z = m[2]
        d = means + (rot.T @ t)[:, None]
        self.Y = _basis(deg, *(d / d.norm(dim=0, keepdim=True)))
        C = (a["sh"].double() if sh is None else sh).view(-1, 3, self.n)
        self.f = (C * self.Y[:, None]).sum(0) + 0.5
        self.mask, self.M = mask, None if M is None else M.double().view(3, 3)
        self.pre = self.f if mask is None else torch.where(mask[None], self.M @ self.f + b.double()[:, None], self.f)
        self.rgb = self.pre.clamp(min=0).T.contiguous()
        limx, limy = 1.3 * 0.5 * W / cam.fx, 1.3 * 0.5 * H / cam.fy
        xc, yc = (m[0] / z).clamp(-limx, limx) * z, (m[1] / z).clamp(-limy, limy) * z
        J0 = torch.stack([cam.fx / z, torch.zeros_like(z), -cam.fx * xc / z ** 2])
        J1 = torch.stack([torch.zeros_like(z), cam.fy / z, -cam.fy * yc / z ** 2])
        p, q = rot.T @ J0, rot.T @ J1
        c = _cov64(a["log_scales"], a["quats"])
        S = [[c[0], c[1], c[2]], [c[1], c[3], c[4]], [c[2], c[4], c[5]]]
        sp = torch.stack([S[i][0] * p[0] + S[i][1] * p[1] + S[i][2] * p[2] for i in range(3)])
        sq = torch.stack([S[i][0] * q[0] + S[i][1] * q[1] + S[i][2] * q[2] for i in range(3)])
        A, B, D = (p * sp).sum(0) + 0.3, (p * sq).sum(0), (q * sq).sum(0) + 0.3
        det = A * D - B * B
        self.sigma = a["opacity"].double()
        self.con = torch.stack([D / det, -B / det, A / det], 1)
        self.uv = torch.stack([cam.fx * m[0] / z + cam.cx, cam.fy * m[1] / z + cam.cy], 1)
        level = 2 * torch.log(255 * self.sigma) + 1 / 64
        ok = (z > cam.znear) & (det > 0) & (255 * self.sigma >= 1)
        e = torch.stack([torch.sqrt((level * A).clamp(min=0)), torch.sqrt((level * D).clamp(min=0))], 1)
        lim = torch.tensor([W - 1.0, H - 1.0], dtype=torch.float64, device=DEV)
        lo = torch.ceil(self.uv - e - 0.5).clamp(min=0)
        hi = torch.minimum(torch.floor(self.uv + e - 0.5), lim)
        ok &= (lo <= hi).all(1)
        self.tx, self.T = (W + 31) // 32, 32
        idx = torch.nonzero(ok).squeeze(1)
        idx = idx[torch.sort(z[idx].float(), stable=True).indices]
        t0, t1 = (lo[idx] / 32).long(), (hi[idx] / 32).long()
        wd = t1[:, 0] - t0[:, 0] + 1
        cnt = wd * (t1[:, 1] - t0[:, 1] + 1)
        own = torch.repeat_interleave(torch.arange(idx.numel(), device=DEV), cnt)
        k = torch.arange(own.numel(), device=DEV) - (torch.cumsum(cnt, 0) - cnt)[own]
        tile = (t0[own, 1] + k // wd[own]) * self.tx + t0[own, 0] + k % wd[own]
        tile, perm = torch.sort(tile, stable=True)
        self.lists = idx[own[perm]]
        nt = self.tx * ((H + 31) // 32)
        self.ends = torch.cumsum(torch.bincount(tile, minlength=nt), 0).tolist()

    def tiles(self):
        W, H, at = self.cam.width, self.cam.height, 0
        for t, end in enumerate(self.ends):
            x0, y0 = t % self.tx * 32, t // self.tx * 32
            yield slice(y0, min(H, y0 + 32)), slice(x0, min(W, x0 + 32)), self.lists[at:end]
            at = end

    def blend(self, ys, xs, idx):
        py = (torch.arange(ys.start, ys.stop, device=DEV, dtype=torch.float64) + 0.5)[:, None].expand(-1, xs.stop - xs.start).reshape(-1, 1)
        px = (torch.arange(xs.start, xs.stop, device=DEV, dtype=torch.float64) + 0.5)[None, :].expand(ys.stop - ys.start, -1).reshape(-1, 1)
        uv, con = self.uv[idx], self.con[idx]
        dx, dy = px - uv[:, 0], py - uv[:, 1]
        G = torch.exp(-0.5 * (con[:, 0] * dx * dx + con[:, 2] * dy * dy) - con[:, 1] * dx * dy)
        raw = self.sigma[idx] * G
        al = torch.where(raw >= 1 / 255, raw.clamp(max=0.99), torch.zeros_like(raw))
        lg = torch.log1p(-al)
        Tn = torch.exp(torch.cumsum(lg, 1))
        on = (Tn >= 1e-4) & (al > 0)
        return G, raw, al, Tn * torch.exp(-lg) * on, on, torch.where(on, Tn, torch.ones_like(Tn))

    def image(self):
        img = torch.zeros(self.cam.height, self.cam.width, 3, dtype=torch.float64, device=DEV)
        for ys, xs, idx in self.tiles():
            if idx.numel():
                _, _, al, T, _, _ = self.blend(ys, xs, idx)
                img[ys, xs] = ((al * T) @ self.rgb[idx]).view(ys.stop - ys.start, -1, 3)
        return img

    def backward(self, g):
        """(dL/dopacity, colour gradient before the clamp and the recolour [3][n], dL/dM)."""
        dsig = torch.zeros(self.n, dtype=torch.float64, device=DEV)
        drgb = torch.zeros(self.n, 3, dtype=torch.float64, device=DEV)
        for ys, xs, idx in self.tiles():
            if not idx.numel():
                continue
            G, raw, al, T, on, _ = self.blend(ys, xs, idx)
            gp = g[ys, xs].reshape(-1, 3)
            s = gp @ self.rgb[idx].T
            ws = al * T * s
            behind = ws.sum(1, keepdim=True) - torch.cumsum(ws, 1)
            dal = torch.where(on & (raw < 0.99), T * s - behind / (1 - al), torch.zeros_like(s))
            dsig.index_add_(0, idx, (dal * G).sum(0))
            drgb.index_add_(0, idx, (al * T).T @ gp)
        gh = torch.where(self.pre > 0, drgb.T, torch.zeros_like(self.pre))
        gc, dM = gh, torch.zeros(9, dtype=torch.float64, device=DEV)
        if self.mask is not None:
            gc = torch.where(self.mask[None], self.M.T @ gh, gh)
            dM = ((gh * self.mask) @ self.f.T).reshape(9)
        return dsig, gc, dM


def _blur64(x):
    r = torch.arange(-5, 6, dtype=torch.float64)
    g = torch.exp(-r * r / (2 * 1.5 * 1.5))
    g = (g / g.sum()).tolist()
    h, w = x.shape[:2]
    p = torch.nn.functional.pad(x, (0, 0, 5, 5, 5, 5))
    p = sum(g[k] * p[:, k:k + w] for k in range(11))
    return sum(g[k] * p[k:k + h] for k in range(11))


def _loss64(y, t):
    """(L1 term, SSIM term, gradient of their sum)."""
    y = y.double().detach().requires_grad_(True)
    t = t.double()
    my, mt = _blur64(y), _blur64(t)
    vy, vt, vyt = _blur64(y * y) - my * my, _blur64(t * t) - mt * mt, _blur64(y * t) - my * mt
    c1, c2 = 0.01 ** 2, 0.03 ** 2
    S = (2 * my * mt + c1) * (2 * vyt + c2) / ((my * my + mt * mt + c1) * (vy + vt + c2))
    l1, l2 = (1 - LAMBDA) * (y - t).abs().mean(), LAMBDA * (1 - S.mean())
    (l1 + l2).backward()
    return l1.detach().reshape(1), l2.detach().reshape(1), y.grad


def exact(c, seed):
    kind = c["kind"]
    if kind == "loss":
        a, b, g = _loss64(_picture(seed, c["h"], c["w"], 1), _picture(seed, c["h"], c["w"], 2))
        return dict(grad=g, loss=a + b)
    if kind == "cloud":
        p, k = _cloud(seed, c["n"]).double(), c["k"]
        n = p.shape[1]
        dist = torch.empty(n, dtype=torch.float64, device=DEV)
        step = max(1, 300_000_000 // n)
        for i in range(0, n, step):
            d = sum((p[j][None] - p[j, i:i + step][:, None]) ** 2 for j in range(3))
            dist[i:i + step] = torch.sqrt(torch.topk(d, k + 1, largest=False, sorted=True).values[:, 1:]).mean(1)
        return dict(clean=None, kept=None, count=None, dist=dist)
    if kind == "batch":
        sizes = [int(x) for x in c["sizes"].split(",")]
        res = [tuple(int(v) for v in x.split("x")) for x in c["res"].split(",")]
        if sum(sizes) * len(res) > 6_000_000:
            return None
        M, b = _edit(seed)
        out = []
        for k, cam in enumerate(_cameras(seed, res * len(sizes))):
            si = k // len(res)
            if k % len(res) == 0:
                a = _arrays(seed, sizes[si], c["deg"], c["storage"], si)
            out.append(Render64(a, cam, c["deg"], mask=_mask64(seed, a, cam), M=M, b=b).image())
        return out
    st = c.get("storage", "f32")
    a = _arrays(seed, c["n"], c["deg"], st)
    M, b = _edit(seed)
    if kind == "bake":
        cam = _cameras(seed, [(1920, 1080)])[0]
        sh = _recolor64(a["sh"].double(), _mask64(seed, a, cam), M, b)
        return dict(cov=torch.stack(_cov64(a["log_scales"], a["quats"])), mask=None, count=None, sh=sh)
    w, h = c["w"], c["h"]
    cams = _cameras(seed, [(w, h)] * c.get("views", 2 if kind == "select" else 1))
    cam = cams[0]
    if kind == "frame":
        mask = _mask64(seed, a, cam)
        if c["edit"] == "recolor":
            sh = _recolor64(a["sh"].double(), mask, M, b)
            # the frame draws the stored coefficients
            return dict(sh=sh, image=Render64(a, cam, c["deg"], sh=sh.to(DTYPE[st]).double()).image())
        if c["edit"] == "none":
            return dict(image=Render64(a, cam, c["deg"]).image())
        return dict(image=Render64(a, cam, c["deg"], mask=mask, M=M, b=b).image())
    if kind == "diff":
        mask = _mask64(seed, a, cam)
        images, loss, dop, dc, dM = [], [], 0, 0, 0
        for k, cam in enumerate(cams):
            r = Render64(a, cam, c["deg"], mask=mask, M=M, b=b)
            y = r.image()
            d = y - _picture(seed, h, w, 8 + k).double()
            images.append(y)
            loss.append(d.square().mean())
            x = r.backward(2 * d / d.numel())
            dop, dc, dM = dop + x[0], dc + Y00 * x[1], dM + x[2]
        return dict(images=images, loss=torch.stack(loss), dop=dop, ddc=dc, dM=dM)
    if kind == "refit":
        r = Render64(a, cam, c["deg"])
        y = r.image()
        l1, l2, g = _loss64(y, _picture(seed, h, w, 8))
        dop, gc, _ = r.backward(g)
        dsh = (r.Y[:, None] * gc[None]).reshape(-1, c["n"])
        mo = _moments(_gen(seed, 3), a["sh"].shape[0], c["n"])
        b1, b2, lr = float(np.float32(BETA1)), float(np.float32(BETA2)), float(np.float32(LR))
        m = b1 * mo["m"].double() + (1 - b1) * dsh
        v = b2 * mo["v"].double() + (1 - b2) * dsh * dsh
        sh = a["sh"].double() - lr * (m / (1 - b1 ** STEP)) / (torch.sqrt(v / (1 - b2 ** STEP)) + EPS)
        out = dict(image=y, loss=torch.cat([l1 + l2, torch.zeros_like(l1)] if c["fused"] else [l1, l2]), grad=g, dop=dop, sh=sh,
                   m=m, v=v)
        return out if c["fused"] else dict(out, dsh=dsh)
    return dict(image=Render64(a, cam, c["deg"]).image())
