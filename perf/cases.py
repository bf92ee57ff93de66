"""The work that users of gsblend have it do, as cases to be timed: what goes in, one pass through
the public entry points, and what a plain 64-bit evaluation of the same inputs gives.

Four kinds of pass:

* ``frame``: one image through ``api.bin_tiles`` and the differentiable blend. ``path`` "render"
  is the forward alone, "autograd" a training step (``autograd.blend`` and its backward).
* ``loop``: the same frame as a training or serving loop calls it that keeps its workspace and
  buffers: ``bin_count`` + ``bin_fill``, ``pack_gaussians``, the packed forward and backward
  (``path`` "packed"), or the deterministic backward (``path`` "deterministic").
* ``views``: a batch of views of uneven size in one ``api.BatchedViews`` step.
* ``project``: 3D Gaussians through ``api.project``.

The scenes follow the laws of the repository's synthetic scenes (uniform means, log-normal or
log-uniform axes, uniform or Beta(2, 2) opacity, upstream gradient N(0, 1)), drawn on the GPU from
the seed alone.
"""
import math

import torch

from paper_2604_02120_amd import api
from paper_2604_02120_amd.autograd import blend

BG = (0.1, 0.2, 0.3)
RESOLUTIONS = ((854, 480), (1280, 720), (1920, 1080))
TILE = 16


def listed():
    def frame(name, width, height, n, prec, path, sigma="lognormal", median=2.0,
              opacity="uniform", bins="rect", kind="frame"):
        return dict(name=name, kind=kind, width=width, height=height, n=n, prec=prec, path=path,
                    sigma=sigma, median=median, opacity=opacity, bins=bins)

    return [
        # the smallest training step: a crop or a unit-test scene, where launches and host time count
        frame("train_64x64_2k_fp16", 64, 64, 2_000, "fp16", "autograd", sigma="loguniform"),
        # a small preview of odd size, forward only, plain FP32 form
        frame("render_333x217_20k_fp32", 333, 217, 20_000, "fp32", "render"),
        # rendering one 720p frame from scratch
        frame("render_720p_500k_fp16", 1280, 720, 500_000, "fp16", "render"),
        # one training step of a 720p view through autograd, nothing kept between steps
        frame("train_720p_500k_bf16", 1280, 720, 500_000, "bf16", "autograd"),
        # 1080p training loop with kept buffers, in the FP16 GEMM form and in the plain FP32 form
        frame("loop_1080p_1m_fp16", 1920, 1080, 1_000_000, "fp16", "packed", kind="loop"),
        frame("loop_1080p_1m_fp32", 1920, 1080, 1_000_000, "fp32", "packed", kind="loop"),
        # the largest frame: 4K, with the 3-sigma binning and with the opacity-aware one
        frame("loop_4k_3m_bf16", 3840, 2160, 3_000_000, "bf16", "packed", median=3.0,
              opacity="beta22", kind="loop"),
        frame("loop_4k_3m_visible_bf16", 3840, 2160, 3_000_000, "bf16", "packed", median=3.0,
              opacity="beta22", bins="visible", kind="loop"),
        # a reproducible training step at an odd size
        frame("loop_997x613_150k_det_bf16", 997, 613, 150_001, "bf16", "deterministic", kind="loop"),
        # a training batch of 8 views of uneven size
        dict(name="views_8x300k_fp16", kind="views", views=8, n=300_000, prec="fp16"),
        # preprocessing of a whole degree-3 scene, and of a small degree-1 one
        dict(name="project_1m_sh3", kind="project", width=1920, height=1080, n=1_000_000, coeffs=16),
        dict(name="project_4097_sh1", kind="project", width=333, height=217, n=4_097, coeffs=4),
    ]


def draw(rng):
    """One more case of the ranges above; sizes over their logarithm, odd ones among them."""
    kind = rng.choice(("frame", "frame", "loop", "loop", "loop", "views", "project"))
    if kind == "project":
        return dict(kind=kind, width=rng.randrange(64, 1921), height=rng.randrange(64, 1081),
                    n=_log_int(rng, 1_000, 1_000_000), coeffs=rng.choice((1, 4, 9, 16)))
    if kind == "views":
        return dict(kind=kind, views=rng.randrange(2, 9), n=_log_int(rng, 20_000, 300_000),
                    prec=rng.choice(("fp16", "bf16", "fp32")))
    pixels = _log_int(rng, 64 * 64, 1920 * 1080 if kind == "frame" else 3840 * 2160)
    aspect = math.exp(rng.uniform(math.log(0.6), math.log(2.4)))
    width = max(17, int(math.sqrt(pixels * aspect)))
    height = max(17, pixels // width)
    case = dict(kind=kind, width=width, height=height,
                n=max(100, min(3_000_000, int(width * height * rng.uniform(0.15, 0.36)))),
                prec=rng.choice(("fp16", "bf16", "fp32")), sigma="lognormal",
                median=rng.choice((2.0, 3.0)), opacity=rng.choice(("uniform", "beta22")),
                bins=rng.choice(("rect", "rect", "visible")))
    if kind == "frame":
        case["path"] = rng.choice(("render", "autograd"))
    else:
        # the deterministic backward's workspace grows with the list: frames up to 1080p
        small = width * height <= 1920 * 1080
        case["path"] = rng.choice(("packed", "packed", "deterministic")) if small else "packed"
    return case


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# ----------------------------------------------------------------------------------- inputs
def _scene(width, height, n, sigma, median, opacity, seed):
    """One scene and its upstream gradient, FP32 on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    opts = dict(device="cuda", dtype=torch.float64, generator=g)
    x = torch.rand(n, **opts) * width
    y = torch.rand(n, **opts) * height
    theta = torch.rand(n, **opts) * math.pi
    if sigma == "loguniform":
        s = torch.exp(torch.rand(n, 2, **opts) * math.log(16.0) + math.log(0.5))
    else:
        s = torch.exp(torch.randn(n, 2, **opts) * 0.932 + math.log(median)).clamp_(0.5, 64.0)
    if opacity == "beta22":      # the middle of three uniforms is Beta(2, 2)
        o = torch.rand(n, 3, **opts).median(dim=1).values * 0.99
    else:
        o = torch.rand(n, **opts) * 0.94 + 0.05
    rgb = torch.rand(n, 3, **opts)
    depth = torch.rand(n, **opts) * 99.0 + 1.0
    c, sn = torch.cos(theta), torch.sin(theta)
    i1, i2 = s[:, 0] ** -2, s[:, 1] ** -2
    conics = torch.stack([c * c * i1 + sn * sn * i2, c * sn * (i1 - i2), sn * sn * i1 + c * c * i2], 1)
    f32 = lambda t: t.to(torch.float32).contiguous()  # noqa: E731
    return dict(width=width, height=height, means2d=f32(torch.stack([x, y], 1)), conics=f32(conics),
                opacity=f32(o), colors=f32(rgb), depths=f32(depth),
                radii=torch.ceil(3.0 * s.amax(dim=1)).to(torch.int32),
                dloss=torch.randn(3, height, width, device="cuda", generator=g))


def _case_scene(case, seed):
    return _scene(case["width"], case["height"], case["n"], case["sigma"], case["median"],
                  case["opacity"], seed)


def _view_scenes(case, seed):
    return [_scene(*RESOLUTIONS[v % len(RESOLUTIONS)], case["n"], "lognormal", 2.0, "uniform",
                   seed * 1000 + v) for v in range(case["views"])]


def _scene3d(case, seed):
    """3D Gaussians in front of a camera that is turned a little, with a camera to match."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    n, W, H, K = case["n"], case["width"], case["height"], case["coeffs"]
    opts = dict(device="cuda", dtype=torch.float64, generator=g)
    f = 1000.0
    u, v = torch.rand(n, **opts) * W, torch.rand(n, **opts) * H
    z = torch.rand(n, **opts) * 18.0 + 2.0
    sig = torch.exp(torch.randn(n, 3, **opts) * 0.932 + math.log(2.0)).clamp_(0.5, 64.0)
    quats = torch.nn.functional.normalize(torch.randn(n, 4, **opts), dim=1)
    sh = torch.randn(n, K, 3, **opts) * 0.15
    sh[:, 0] = torch.rand(n, 3, **opts) * 3.5 - 1.75
    a = 0.3
    R = torch.tensor([[math.cos(a), 0.0, -math.sin(a)], [0.0, 1.0, 0.0],
                      [math.sin(a), 0.0, math.cos(a)]], dtype=torch.float32).double()
    t = torch.tensor([0.25, -0.5, 1.0], dtype=torch.float64)
    pc = torch.stack([(u - W / 2.0) / f * z, (v - H / 2.0) / f * z, z], 1)
    means = (pc - t.cuda()) @ R.cuda()
    f32 = lambda q: q.to(torch.float32).contiguous()  # noqa: E731
    camera = dict(R=R.tolist(), t=t.tolist(), fx=f, fy=f, cx=W / 2.0, cy=H / 2.0, width=W, height=H,
                  near=0.2)
    return dict(means3d=f32(means), scales=f32(sig * (z / f)[:, None]), quats=f32(quats),
                sh=f32(sh), camera=camera)


def prepare(case, seed):
    if case["kind"] == "project":
        s = _scene3d(case, seed)
        s["camera"] = api.camera_struct(**s["camera"])
        return dict(case=case, **s)
    if case["kind"] == "views":
        scenes = _view_scenes(case, seed)
        views = api.BatchedViews(scenes, prec=case["prec"], bg=BG)
        for view, scene in zip(views.views, scenes):
            view["dL_dimage"].copy_(scene["dloss"])
        return dict(case=case, views=views)
    s = _case_scene(case, seed)
    state = dict(case=case, scene=s)
    if case["kind"] == "frame":
        if case["path"] == "autograd":
            for k in ("means2d", "conics", "opacity", "colors"):
                s[k].requires_grad_(True)
        return state
    # a loop's kept buffers: workspace and list for the pair count, outputs, records, gradients
    W, H, n = case["width"], case["height"], case["n"]
    count = api.bin_count(s["means2d"], s["radii"], W, H, api.BinWorkspace(n, 0, W, H),
                          conics=s["conics"], opacity=s["opacity"], mode=case["bins"])
    pairs = int(count.item())
    gx, gy = api.grid(W, H)
    f32 = dict(device="cuda", dtype=torch.float32)
    i32 = dict(device="cuda", dtype=torch.int32)
    state.update(
        ws=api.BinWorkspace(n, pairs, W, H), point_list=torch.empty(pairs, **i32),
        ranges=torch.empty((gx * gy, 2), **i32), records=torch.empty((n, 12), **f32),
        fwd=(torch.empty((3, H, W), **f32), torch.empty((H, W), **f32), torch.empty((H, W), **i32)),
        bwd=(torch.empty((n, 2), **f32), torch.empty((n, 3), **f32), torch.empty((n,), **f32),
             torch.empty((n, 3), **f32)))
    if case["path"] == "deterministic":
        state["det"] = api.DetWorkspace(n, pairs, device="cuda")
    return state


# ----------------------------------------------------------------------------------- one pass
def run(state):
    # The sorted list itself (its length depends on the seed) is not among the outputs: the images,
    # positions and gradients are read off it, and the ranges are its shape.
    case = state["case"]
    kind = case["kind"]
    if kind == "project":
        return api.project(state["means3d"], state["scales"], state["quats"], state["sh"],
                           state["camera"])
    if kind == "views":
        views = state["views"]
        views.step()
        return [[v["image"], v["final_T"], v["last_contrib"], v["dL_dmeans2d"], v["dL_dconics"],
                 v["dL_dopacity"], v["dL_dcolors"], v["ranges"]]
                for v in views.views]
    s, W, H, prec = state["scene"], case["width"], case["height"], case["prec"]
    m, c, o, col = s["means2d"], s["conics"], s["opacity"], s["colors"]
    if kind == "frame":
        plist, ranges = api.bin_tiles(m.detach(), s["radii"], s["depths"], W, H, conics=c.detach(),
                                      opacity=o.detach(), mode=case["bins"])
        if case["path"] == "render":
            return [*api.blend_forward(m, c, o, col, ranges, plist, W, H, BG, prec), ranges]
        image, final_T, last = blend(m, c, o, col, ranges, plist, W, H, BG, prec)
        grads = torch.autograd.grad(image, (m, c, o, col), s["dloss"])
        return [image.detach(), final_T, last, *grads, ranges]
    plist, ranges = state["point_list"], state["ranges"]
    api.bin_count(m, s["radii"], W, H, state["ws"], conics=c, opacity=o, mode=case["bins"])
    status = api.bin_fill(m, s["radii"], s["depths"], W, H, state["ws"], plist, ranges, conics=c,
                          opacity=o, mode=case["bins"])
    rec = api.pack_gaussians(m, c, o, col, out=state["records"])
    image, final_T, last = api.blend_forward_packed(rec, ranges, plist, W, H, BG, prec,
                                                    out=state["fwd"])
    if case["path"] == "deterministic":
        grads = api.blend_backward_deterministic(rec, ranges, plist, W, H, final_T, last,
                                                 s["dloss"], BG, prec, ws=state["det"],
                                                 out=state["bwd"])
    else:
        grads = api.blend_backward_packed(rec, ranges, plist, W, H, final_T, last, s["dloss"], BG,
                                          prec, out=state["bwd"])
    return [image, final_T, last, *grads, ranges, status]


# ----------------------------------------------------------------------------------- its work
def work(case):
    """Inputs read once, outputs written once. Operations of a blend: those of the blended pairs
    (26 forward, 55 backward, each add, multiply, compare and exp one), whose number per pixel is
    estimated from the scene's law: half the layers that cover a pixel, and at most 70, where the
    pixel is opaque."""
    kind, n = case["kind"], case["n"]
    if kind == "project":
        return dict(bytes=n * (40 + 12 * case["coeffs"] + 40), flops=n * (250 + 6 * case["coeffs"]))
    if kind == "views":
        area = 2.0 * math.pi * 4.8 * 2.0 ** 2 * math.exp(0.932 ** 2)
        sizes = [RESOLUTIONS[v % len(RESOLUTIONS)] for v in range(case["views"])]
        each = [_frame_work(w * h, n, area, 5.9, True) for w, h in sizes]
        return {k: sum(e[k] for e in each) for k in ("bytes", "flops")}
    if case["sigma"] == "loguniform":
        area = 2.0 * math.pi * 4.8 * (7.5 / math.log(16.0)) ** 2
        reach = 3.0 * 4.5
    else:
        area = 2.0 * math.pi * 4.8 * case["median"] ** 2 * math.exp(0.932 ** 2)
        reach = 3.0 * 1.9 * case["median"]
    tiles = ((2.0 * reach + TILE) / TILE) ** 2
    return _frame_work(case["width"] * case["height"], n, area, tiles, case["path"] != "render")


def _frame_work(pixels, n, area, tiles, backward):
    blended = pixels * min(70.0, 0.5 * area * n / pixels)
    bytes_ = n * (4 * 9 + 4 + 4) + 4 * n * tiles + pixels * 20 + pixels / 32
    flops = 26 * blended
    if backward:
        bytes_ += pixels * 20 + n * 4 * 9
        flops += 55 * blended
    return dict(bytes=int(bytes_), flops=int(flops))


# ----------------------------------------------------------------------------------- 64 bits
def exact(case, seed):
    """The same outputs in FP64: images and transmittances, gradients, projections. Lists, ranges
    and positions within them are whole numbers and have no entry here."""
    if case["kind"] == "project":
        return _exact_project(_scene3d(case, seed), case)
    if case["kind"] == "views":
        out = []
        for s in _view_scenes(case, seed):
            image, T, grads = _exact_frame(s, True)
            out.append([image, T, None, *grads, None])
        return out
    s = _case_scene(case, seed)
    image, T, grads = _exact_frame(s, case["path"] != "render")
    if case["kind"] == "loop":
        return [image, T, None, *grads, None, None]
    return [image, T, None, *(grads or ()), None]


def _pairs(s):
    """(Gaussian of every pair, first pair and number of pairs of every tile), pairs ordered by
    (tile, depth, index); the 3-sigma square (the opacity-aware rule drops only pairs that the
    blend skips)."""
    W, H = s["width"], s["height"]
    gx, gy = (W + TILE - 1) // TILE, (H + TILE - 1) // TILE
    order = torch.sort(s["depths"], stable=True).indices
    xy = s["means2d"][order].double()
    r = s["radii"][order].double()
    lo = torch.floor((xy - r[:, None]) / TILE)
    hi = torch.floor((xy + r[:, None] + TILE - 1) / TILE)
    lim = torch.tensor([gx, gy], dtype=torch.float64, device=xy.device)
    lo, hi = lo.clamp_min(0).minimum(lim).long(), hi.clamp_min(0).minimum(lim).long()
    wh = (hi - lo).clamp_min(0)
    cnt = wh[:, 0] * wh[:, 1]
    who = torch.repeat_interleave(torch.arange(len(cnt), device=xy.device), cnt)
    k = torch.arange(len(who), device=xy.device) - (torch.cumsum(cnt, 0) - cnt)[who]
    w = wh[:, 0][who]
    tile = ((lo[:, 1][who] + torch.div(k, w, rounding_mode="floor")) * gx + lo[:, 0][who] + k % w)
    tile, perm = torch.sort(tile.int(), stable=True)
    number = torch.bincount(tile.long(), minlength=gx * gy)
    return order[who[perm]], torch.cumsum(number, 0) - number, number


def _exact_frame(s, backward):
    W, H = s["width"], s["height"]
    gx, gy = (W + TILE - 1) // TILE, (H + TILE - 1) // TILE
    dev = s["means2d"].device
    d64 = dict(device=dev, dtype=torch.float64)
    gauss, first, number = _pairs(s)
    n = len(s["opacity"])
    attr = torch.cat([s["means2d"].double(), s["conics"].double(), s["opacity"].double()[:, None],
                      s["colors"].double()], 1)
    bg = torch.tensor(BG, **d64)
    # outputs padded to whole tiles, [tile][pixel of the tile]
    image = torch.empty((gx * gy, TILE * TILE, 3), **d64)
    final = torch.empty((gx * gy, TILE * TILE), **d64)
    if backward:
        up = torch.zeros((3, gy * TILE, gx * TILE), **d64)
        up[:, :H, :W] = s["dloss"].double()
        up = up.view(3, gy, TILE, gx, TILE).permute(1, 3, 2, 4, 0).reshape(gx * gy, TILE * TILE, 3)
        sums = torch.zeros((n, 9), **d64)
    px = torch.arange(TILE, **d64).repeat(TILE)
    py = torch.arange(TILE, **d64).repeat_interleave(TILE)
    by_len = torch.sort(number, descending=True)
    lens, tiles = by_len.values.tolist(), by_len.indices
    at = 0
    while at < len(lens):
        L = max(lens[at], 1)
        take = min(len(lens) - at, max(1, (1 << 27) // (L * TILE * TILE)))
        t = tiles[at:at + take]
        at += take
        j = torch.arange(L, device=dev)
        has = j < number[t][:, None]                                  # [t][L]
        if len(gauss):
            g = gauss[(first[t][:, None] + j).clamp_max(len(gauss) - 1)]
        else:
            g = torch.zeros_like(has, dtype=torch.long)
        a = attr[g] if n else torch.zeros((*g.shape, 9), **d64)
        dx = a[..., 0:1] - (px + (t % gx)[:, None, None] * TILE)      # [t][L][256]
        dy = a[..., 1:2] - (py + torch.div(t, gx, rounding_mode="floor")[:, None, None] * TILE)
        power = -0.5 * (a[..., 2:3] * dx * dx + a[..., 4:5] * dy * dy) - a[..., 3:4] * dx * dy
        raw = a[..., 5:6] * torch.exp(power.clamp_max(0.0))
        alpha = raw.clamp_max(0.99)
        alpha = torch.where(has[..., None] & (alpha >= 1.0 / 255.0), alpha, 0.0)
        after = torch.cumprod(1.0 - alpha, 1)
        alpha = torch.where(after >= 1e-4, alpha, 0.0)                # T only falls: a stop is final
        after = torch.cumprod(1.0 - alpha, 1)
        before = after / (1.0 - alpha)
        w = alpha * before
        T = after[:, -1]
        col = a[..., 6:9]
        image[t] = torch.matmul(w.transpose(1, 2).contiguous(), col) + T[..., None] * bg
        final[t] = T
        if not backward:
            continue
        u = up[t]                                                     # [t][256][3]
        cg = torch.matmul(col, u.transpose(1, 2).contiguous())        # [t][L][256]
        wcg = w * cg
        behind = wcg.sum(1, keepdim=True) - torch.cumsum(wcg, 1) + (T * (u @ bg))[:, None]
        da = before * cg - behind / (1.0 - alpha)
        da = torch.where((alpha > 0.0) & (raw < 0.99), alpha * da, 0.0)   # dL/dpower
        dg = torch.where(power <= 0.0, da, 0.0)
        part = torch.stack([(dg * dx * dx).sum(-1), (dg * dx * dy).sum(-1), (dg * dy * dy).sum(-1),
                            (dg * dx).sum(-1), (dg * dy).sum(-1), da.sum(-1)], -1)
        part = torch.cat([part, torch.matmul(w, u)], -1)
        sums.index_add_(0, g.reshape(-1), part.reshape(-1, 9))

    def untile(v):
        c = v.shape[-1] if v.dim() == 3 else 1
        v = v.view(gy, gx, TILE, TILE, c).permute(4, 0, 2, 1, 3).reshape(c, gy * TILE, gx * TILE)
        return v[:, :H, :W].contiguous()

    out = untile(image), untile(final)[0]
    if not backward:
        return (*out, None)
    A, B, C, o = attr[:, 2], attr[:, 3], attr[:, 4], attr[:, 5]
    sx, sy = sums[:, 3], sums[:, 4]
    grads = (torch.stack([-(A * sx + B * sy), -(B * sx + C * sy)], 1),
             torch.stack([-0.5 * sums[:, 0], -sums[:, 1], -0.5 * sums[:, 2]], 1),
             sums[:, 5] / o, sums[:, 6:9].contiguous())
    return (*out, grads)


def _exact_project(s, case):
    cam = s["camera"]
    dev = s["means3d"].device
    d64 = dict(device=dev, dtype=torch.float64)
    m, sc, q = s["means3d"].double(), s["scales"].double(), s["quats"].double()
    R = torch.tensor(cam["R"], **d64).float().double()
    t = torch.tensor(cam["t"], **d64).float().double()
    fx, fy, cx, cy, W, H = (cam[k] for k in ("fx", "fy", "cx", "cy", "width", "height"))
    p = m @ R.T + t
    z = p[:, 2]
    xz, yz = p[:, 0] / z, p[:, 1] / z
    u, v = fx * xz + cx, fy * yz + cy
    w, x, y, k = torch.nn.functional.normalize(q, dim=1).unbind(1)
    rot = torch.stack([1 - 2 * (y * y + k * k), 2 * (x * y - w * k), 2 * (x * k + w * y),
                       2 * (x * y + w * k), 1 - 2 * (x * x + k * k), 2 * (y * k - w * x),
                       2 * (x * k - w * y), 2 * (y * k + w * x), 1 - 2 * (x * x + y * y)],
                      1).view(-1, 3, 3)
    M = rot * sc[:, None, :]
    lx, ly = 1.3 * W / (2.0 * fx), 1.3 * H / (2.0 * fy)
    zero = torch.zeros_like(z)
    J = torch.stack([fx / z, zero, -fx * xz.clamp(-lx, lx) / z,
                     zero, fy / z, -fy * yz.clamp(-ly, ly) / z], 1).view(-1, 2, 3)
    P = torch.matmul(torch.matmul(J, R), M)
    a = (P[:, 0] ** 2).sum(1) + 0.3
    b = (P[:, 0] * P[:, 1]).sum(1)
    c = (P[:, 1] ** 2).sum(1) + 0.3
    det = a * c - b * b
    mid = 0.5 * (a + c)
    lmax = mid + torch.sqrt((mid * mid - det).clamp_min(0.1))
    r = torch.ceil(3.0 * torch.sqrt(lmax))
    gx, gy = (W + TILE - 1) // TILE, (H + TILE - 1) // TILE
    span = lambda q, g: (torch.floor((q + r + TILE - 1) / TILE).clamp(0, g)  # noqa: E731
                         > torch.floor((q - r) / TILE).clamp(0, g))
    keep = (z > cam["near"]) & (det > 0) & span(u, gx) & span(v, gy)
    d = torch.nn.functional.normalize(m + t @ R, dim=1)
    Y = _harmonics(d, case["coeffs"])
    col = (0.5 + (Y[:, :, None] * s["sh"].double()).sum(1)).clamp_min(0.0)
    mask = lambda v: torch.where(keep.view(-1, *[1] * (v.dim() - 1)), v, 0.0)  # noqa: E731
    return [mask(torch.stack([u, v], 1)), mask(torch.stack([c, -b, a], 1) / det[:, None]), mask(z),
            None, mask(col)]


def _harmonics(d, K):
    """Real spherical harmonics of degree <= 3 at unit directions, order (l, m = -l..l)."""
    x, y, z = d.unbind(1)
    pi = math.pi
    c1, c2 = math.sqrt(3 / (4 * pi)), math.sqrt(15 / pi)
    c3, c4 = math.sqrt(35 / (2 * pi)) / 4, math.sqrt(105 / pi)
    c5, c6 = math.sqrt(21 / (2 * pi)) / 4, math.sqrt(7 / pi) / 4
    rows = [torch.full_like(x, 0.5 / math.sqrt(pi)), -c1 * y, c1 * z, -c1 * x,
            c2 / 2 * x * y, -c2 / 2 * y * z, math.sqrt(5 / pi) / 4 * (2 * z * z - x * x - y * y),
            -c2 / 2 * x * z, c2 / 4 * (x * x - y * y),
            -c3 * y * (3 * x * x - y * y), c4 / 2 * x * y * z, -c5 * y * (4 * z * z - x * x - y * y),
            c6 * z * (2 * z * z - 3 * x * x - 3 * y * y), -c5 * x * (4 * z * z - x * x - y * y),
            c4 / 4 * z * (x * x - y * y), -c3 * x * (x * x - 3 * y * y)]
    return torch.stack(rows[:K], 1)
