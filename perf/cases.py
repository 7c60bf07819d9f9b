"""The work this framework is measured on: what its users run, from the smallest call to the
largest, through the public entry points (the trainer, the autograd wrappers and the C-ABI
binding).

A case names the way of use ("kind") and its sizes:

  step      one iteration of the trainer (render, loss, gate, backward, Adam in one call)
  skip      the same iteration when the gate skips the backward
  eval      a held-out view rendered, and its loss
  autograd  render and loss through torch.autograd, gradients of every parameter
  batch     a minibatch of views in one launch: render, losses, backward, plain Adam step
  loss      the photometric loss of an image and its gradient
  densify   one clone / split / prune step
  grow      an iteration of the densification phase with its gradient statistic

Scenes, cameras and their ranges are those of paper_2603_08997_amd.scenes (mixture, dense and
tiny scenes, hemisphere and tetrahedron views), drawn on the GPU because the large ones would
take seconds in numpy.
"""
import math

import numpy as np
import torch

from paper_2603_08997_amd import autograd as ag
from paper_2603_08997_amd import scenes as S
from paper_2603_08997_amd import skipgs as sk
from paper_2603_08997_amd import train as T

LAM = 0.2            # weight of the SSIM term
LARGEST = 3_000_000  # Gaussians of the training benchmark


def listed():
    def c(name, kind, n, sh, w, h, views, scene="mixture", option=""):
        return dict(name=name, kind=kind, n=n, sh=sh, width=w, height=h, views=views, scene=scene, option=option)

    return [
        # the smallest training run (unit tests, demos, first experiments): launches and latency count
        c("step_tiny", "step", 1000, 0, 64, 64, 4, "tiny", "gated"),
        # the same scene by a researcher's own torch loop: four views, gradients by autograd
        c("autograd_tiny", "autograd", 1000, 0, 64, 64, 4, "tiny", "keep"),
        # an object-sized scene at an odd image size, low SH degree, workspace kept for the backward
        c("autograd_30k_637x479", "autograd", 30011, 1, 637, 479, 1, "mixture", "keep"),
        # early training: the set still grows, view-space gradients are gathered
        c("grow_300k_980x545", "grow", 300007, 3, 980, 545, 4),
        # quality checks during training and serving of novel views
        c("eval_1M_1245x825", "eval", 1_000_000, 3, 1245, 825, 4),
        # the visible-only optimiser option at an intermediate SH degree
        c("step_visible_1M_1245x825", "step", 1_000_000, 2, 1245, 825, 4, "mixture", "visible"),
        # the loss alone, as a user with a renderer of their own calls it
        c("loss_1600x1060", "loss", 0, 0, 1600, 1060, 1),
        # the training benchmark: every iteration runs its backward ...
        c("step_3M_1600x1060", "step", LARGEST, 3, 1600, 1060, 4, "mixture", "full"),
        # ... and the half of them that the gate skips
        c("skip_3M_1600x1060", "skip", LARGEST, 3, 1600, 1060, 4),
        # a minibatch of eight views of four resolutions in one launch
        c("batch_2M_8views", "batch", 2_000_000, 3, 0, 0, 8),
        # the density step of the growth phase
        c("densify_3M", "densify", LARGEST, 3, 0, 0, 0),
        # high depth complexity, through autograd with the forward run again in the backward
        c("autograd_dense_6M", "autograd", 6_000_000, 3, 1600, 1060, 1, "dense", "recompute"),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["step", "step", "skip", "eval", "autograd", "autograd", "batch", "loss", "densify", "grow"])
    w, sh = log_int(64, 1600), rng.choice([0, 1, 2, 3, 3])
    h = max(48, int(w * rng.uniform(0.5, 0.8)))
    # a set has between a quarter of a Gaussian and two Gaussians for each pixel of its views
    n = min(LARGEST, max(1000, int(w * h * math.exp(rng.uniform(math.log(0.25), math.log(2.0))))))
    views, scene, option = rng.choice([2, 4, 8]), "mixture", ""
    if kind == "step":
        option = rng.choice(["gated", "full", "visible"])
    elif kind == "autograd":
        option = rng.choice(["keep", "recompute"])
        scene = rng.choice(["mixture", "dense"])
        views = rng.choice([1, 1, 2])
    elif kind == "batch":
        n, views, w, h = log_int(100_000, 2_000_000), rng.randint(2, 8), 0, 0
    elif kind == "loss":
        n = sh = 0
        views = 1
    elif kind == "densify":
        n, w, h, views = log_int(5000, LARGEST), 0, 0, 0
    if w and n and n < 5000:
        scene = "tiny"
    return dict(kind=kind, n=n, sh=sh, width=w, height=h, views=views, scene=scene, option=option)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) & 0x7FFFFFFF)
    return g


def _planes(case, seed):
    """Parameter planes [F][stride] of the case's scene."""
    g, n, sh = _gen(seed), case["n"], case["sh"]
    normal = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    uniform = lambda *s: torch.rand(*s, generator=g, device="cuda")  # noqa: E731
    p = torch.zeros(S.n_planes(sh), S.padded_stride(n), device="cuda")
    if case["scene"] == "tiny":
        p[0:3, :n] = 2.0 * uniform(3, n) - 1.0
        log_scale, scale_std, logit, logit_std = -2.2 + math.log(1000 / n) / 3, 0.3, 0.0, 1.0
    else:
        dense = case["scene"] == "dense"
        comp = torch.randint(1 if dense else 0, 3, (n,), generator=g, device="cuda")
        r, th = 6.0 * uniform(n).sqrt(), 2.0 * math.pi * uniform(n)
        disk = torch.stack([r * th.cos(), r * th.sin(), 0.05 * normal(n)])
        sign = torch.where(comp == 1, 1.0, -1.0)
        centre = torch.stack([sign, sign, torch.full_like(sign, 0.5)])
        p[0:3, :n] = torch.where(comp == 0, disk, centre + (0.35 if dense else 0.5) * normal(3, n))
        # smaller sets have larger Gaussians, so that they cover the image
        log_scale = (-3.6 if dense else -4.0) + math.log(max(1.0, 1e6 / n)) / 3
        scale_std, logit, logit_std = 0.5, (-0.45 if dense else 0.0), (1.0 if dense else 1.5)
    p[3:6, :n] = log_scale + scale_std * normal(3, n)
    q = normal(4, n)
    p[6:10, :n] = q / q.norm(dim=0, keepdim=True)
    p[10, :n] = logit + logit_std * normal(n)
    p[11:14, :n] = S.SH_DC_HALF_RANGE * (2.0 * uniform(3, n) - 1.0)
    for j in range(14, p.shape[0]):
        p[j, :n] = 0.05 * normal(n)
    return p


def _perturbed(planes, n, seed):
    """A trainable start: the ground truth plus noise."""
    g, p = _gen(seed), planes.clone()
    for j, s in [(0, 0.02), (1, 0.02), (2, 0.02), (3, 0.1), (4, 0.1), (5, 0.1), (10, 0.5), (11, 0.1), (12, 0.1), (13, 0.1)]:
        p[j, :n] += s * torch.randn(n, generator=g, device="cuda")
    return p


def _cameras(case, seed):
    if case["scene"] == "tiny" and case["views"] == 4:
        return S.tetra_cameras(width=case["width"], height=case["height"])
    if case["kind"] == "batch":
        sizes = [S.BATCH_RESOLUTIONS[k // 2] for k in range(8)][:case["views"]]
        return [S.hemisphere_cameras(1000 * seed + k, 1, w, h)[0] for k, (w, h) in enumerate(sizes)]
    return S.hemisphere_cameras(seed, case["views"], case["width"], case["height"])


def _capacity(planes, case, cams, together):
    """Pair capacity with some room, as a program that has rendered its views once knows it."""
    rp, n, best = sk.RasterParams(), case["n"], 0
    for group in ([cams] if together else [[c] for c in cams]):
        cap = max(4096, 8 * n * len(group))
        rgb = torch.empty(3 * sum(c.width * c.height for c in group), device="cuda")
        for _ in range(3):
            ws = sk.alloc_bytes(sk.forward_workspace_size(rp, n, group, cap))
            sk.clear_status(ws)
            sk.render_forward(planes, n, case["sh"], group, rp, ws, cap, rgb)
            flags, _, need = sk.read_status(ws)
            if not flags & sk.STATUS_PAIR_OVERFLOW:
                break
            cap = int(need * 1.25) + 4096
        best = max(best, need)
    return int(best * 1.25) + 4096


def _moments(planes, n, seed):
    """Adam moments of a run in progress: gradients of the mean losses are around 1e-7."""
    g = _gen(seed)
    m, v = torch.zeros_like(planes), torch.zeros_like(planes)
    for j in range(planes.shape[0]):
        m[j, :n] = 1e-7 * torch.randn(n, generator=g, device="cuda")
        v[j, :n] = (3e-7 * (0.1 + torch.rand(n, generator=g, device="cuda"))) ** 2
    return m, v, torch.full((1,), 1000, dtype=torch.int32, device="cuda")


def _trainer(case, seed):
    n, kind = case["n"], case["kind"]
    truth, cams = _planes(case, seed), _cameras(case, seed)
    cap = _capacity(truth, case, cams, False)
    rp = sk.RasterParams()
    targets = torch.empty(len(cams), 3 * cams[0].width * cams[0].height, device="cuda")
    ws = sk.alloc_bytes(sk.forward_workspace_size(rp, n, [cams[0]], cap))
    sk.clear_status(ws)
    for i, c in enumerate(cams):
        sk.render_forward(truth, n, case["sh"], [c], rp, ws, cap, targets[i])
    planes = _perturbed(truth, n, seed + 1)
    m, v, step = _moments(planes, n, seed + 2)
    gate = None
    if case["option"] == "gated":
        gate = sk.windowed_gate(len(cams))
    elif kind == "skip":
        gate = sk.GateParams(n_views=len(cams), warmup=0, calibrate=False, budget=False, delta=0.02)
    tr = T.Trainer(None, cams, targets, rp, gate, cap + cap // 8, gated=gate is not None, fused=kind != "grow",
                   sequence=np.arange(len(cams)), visible_only=case["option"] == "visible",
                   state=(planes, m, v, step, n, case["sh"]))
    if kind == "skip":  # every view has a loss average above its losses: the gate skips
        for i in range(len(cams)):
            sk.gate_update(gate, tr.gstate, torch.full((1,), i, dtype=torch.int32, device="cuda"),
                           torch.full((1,), 100.0, device="cuda"), tr.gate)
    return tr


def _images(case, seed):
    """A smooth textured picture and a noisy rendering of it, planar."""
    g, w, h = _gen(seed), case["width"], case["height"]
    small = torch.rand(1, 3, max(2, h // 8), max(2, w // 8), generator=g, device="cuda")
    target = torch.nn.functional.interpolate(small, size=(h, w), mode="bicubic", align_corners=False)[0].clamp(0, 1)
    rgb = (target + 0.05 * torch.randn(3, h, w, generator=g, device="cuda")).clamp(0, 1.2)
    return rgb.reshape(-1).contiguous(), target.reshape(-1).contiguous()


def _densify_inputs(case, seed):
    n = case["n"]
    p = sk.DensifyParams(scene_extent=5.0)
    planes = _planes(case, seed)
    m, v, _ = _moments(planes, n, seed + 2)
    g = _gen(seed + 3)
    count = torch.randint(0, 12, (n,), generator=g, device="cuda", dtype=torch.int32)
    grad_sum = count * p.grad_threshold * (0.2 + 0.9 * torch.rand(n, generator=g, device="cuda"))
    return p, planes, m, v, grad_sum, count, torch.randn(n, 2, 3, generator=g, device="cuda")


def prepare(case, seed):
    kind, n = case["kind"], case["n"]
    if kind in ("step", "skip", "grow"):
        tr = _trainer(case, seed)
        s = dict(kind=kind, tr=tr)
        if kind == "grow":
            s.update(turn=0, d_views=torch.arange(len(tr.cams), dtype=torch.int32, device="cuda"),
                     slot=torch.zeros(1, dtype=torch.int32, device="cuda"),
                     grad_sum=torch.zeros(n, device="cuda"),
                     count=torch.zeros(n, dtype=torch.int32, device="cuda"))
        return s
    if kind == "loss":
        rgb, target = _images(case, seed)
        lws = sk.alloc_bytes(sk.loss_workspace_size(case["width"], case["height"]))
        return dict(kind=kind, rgb=rgb, target=target, w=case["width"], h=case["height"], lws=lws,
                    loss=torch.zeros(1, device="cuda"), dl=torch.zeros_like(rgb))
    if kind == "densify":
        p, planes, m, v, grad_sum, count, normals = _densify_inputs(case, seed)
        out = [torch.zeros(planes.shape[0], S.padded_stride(2 * n), device="cuda") for _ in range(3)]
        return dict(kind=kind, p=p, n=n, sh=case["sh"], planes=planes, m=m, v=v, grad_sum=grad_sum, count=count,
                    normals=normals, out=out, ws=sk.alloc_bytes(sk.densify_workspace_size(n)),
                    n_out=torch.zeros(1, dtype=torch.int64, device="cuda"))

    truth, cams = _planes(case, seed), _cameras(case, seed)
    cap, rp = _capacity(truth, case, cams, kind != "eval"), sk.RasterParams()
    group = [cams[0]] if kind == "eval" else cams
    ws = sk.alloc_bytes(sk.forward_workspace_size(rp, n, group, cap))
    sk.clear_status(ws)
    px = [c.width * c.height for c in group]
    target = torch.empty(3 * sum(px), device="cuda")
    sk.render_forward(truth, n, case["sh"], group, rp, ws, cap, target)
    planes = _perturbed(truth, n, seed + 1)
    cap += cap // 8  # the perturbed set's lists differ a little
    s = dict(kind=kind, n=n, sh=case["sh"], cams=cams, rp=rp, cap=cap, planes=planes, target=target, px=px)
    if kind == "autograd":
        s.update(recompute=case["option"] == "recompute")
        s["planes"].requires_grad_(True)
        return s
    s.update(ws=sk.alloc_bytes(sk.forward_workspace_size(rp, n, group, cap)), rgb=torch.zeros(3 * sum(px), device="cuda"),
             loss=torch.zeros(len(group), device="cuda"))
    sk.clear_status(s["ws"])
    if kind == "batch":
        m, v, step = _moments(planes, n, seed + 2)
        s.update(m=m, v=v, step=step, grads=torch.zeros_like(planes), dl=torch.zeros_like(s["rgb"]),
                 adam=sk.AdamParams(lr=sk.default_lrs(case["sh"])),
                 lws=[sk.alloc_bytes(sk.loss_workspace_size(c.width, c.height)) for c in cams])
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def run(s):
    kind = s["kind"]
    if kind in ("step", "skip"):
        tr = s["tr"]
        tr.step()
        return dict(planes=tr.planes, m=tr.m, v=tr.v, rgb=tr.rgb, loss=tr.loss, gate=tr.gate, step=tr.step_count)
    if kind == "grow":
        tr = s["tr"]
        view = s["turn"] % len(tr.cams)
        s["turn"] += 1
        tr.iteration(view, s["d_views"][view:view + 1], s["slot"])
        sk.densify_stats([tr.cams[view]], tr.n, tr.rp, tr.ws, tr.cap, s["grad_sum"], s["count"])
        return dict(planes=tr.planes, m=tr.m, v=tr.v, rgb=tr.rgb, loss=tr.loss, grad_sum=s["grad_sum"], count=s["count"])
    if kind == "loss":
        sk.photometric_loss(s["rgb"], s["target"], s["w"], s["h"], LAM, s["lws"], s["loss"])
        sk.photometric_loss_backward(s["rgb"], s["target"], s["w"], s["h"], LAM, s["lws"], None, s["dl"])
        return dict(loss=s["loss"], dl=s["dl"])
    if kind == "densify":
        sk.densify(s["p"], s["planes"], s["n"], s["sh"], s["m"], s["v"], s["grad_sum"], s["count"], s["normals"],
                   *s["out"], s["ws"], s["n_out"])
        return dict(planes=s["out"][0], m=s["out"][1], v=s["out"][2], n=s["n_out"])
    if kind == "eval":
        c = s["cams"][0]
        sk.render_forward(s["planes"], s["n"], s["sh"], [c], s["rp"], s["ws"], s["cap"], s["rgb"])
        sk.photometric_loss_static(s["rgb"], s["target"], c.width, c.height, LAM, s["loss"])
        return dict(rgb=s["rgb"], loss=s["loss"])
    if kind == "autograd":
        planes = s["planes"]
        planes.grad = None
        rgb = ag.render(planes, s["n"], s["sh"], s["cams"], s["rp"], s["cap"], s["recompute"])
        loss, at = 0.0, 0
        for c, px in zip(s["cams"], s["px"]):
            loss = loss + ag.photometric_loss(rgb[at:at + 3 * px], s["target"][at:at + 3 * px], c.width, c.height, LAM)
            at += 3 * px
        loss.backward()
        return dict(rgb=rgb.detach(), loss=loss.detach(), grad=planes.grad)
    # batch
    sk.render_forward(s["planes"], s["n"], s["sh"], s["cams"], s["rp"], s["ws"], s["cap"], s["rgb"])
    at = 0
    for k, (c, px) in enumerate(zip(s["cams"], s["px"])):
        part = slice(at, at + 3 * px)
        sk.photometric_loss(s["rgb"][part], s["target"][part], c.width, c.height, LAM, s["lws"][k], s["loss"][k:k + 1])
        sk.photometric_loss_backward(s["rgb"][part], s["target"][part], c.width, c.height, LAM, s["lws"][k], None,
                                     s["dl"][part])
        at += 3 * px
    sk.render_backward(s["planes"], s["n"], s["sh"], s["cams"], s["rp"], s["ws"], s["cap"], s["dl"], None, s["grads"])
    sk.adam_step(s["adam"], s["planes"], s["grads"], s["m"], s["v"], s["n"], s["step"])
    return dict(planes=s["planes"], m=s["m"], v=s["v"], rgb=s["rgb"], loss=s["loss"], step=s["step"])


def work(case):
    """Bytes: every input read once, every output written once. Flops: projection and spherical
    harmonics per Gaussian and view, some 60 blended Gaussians per pixel, the two 11-tap filters
    of five moments (and of three maps for the gradient) per pixel and channel."""
    kind, n, f = case["kind"], case["n"], S.n_planes(case["sh"])
    if kind == "batch":
        views, px = case["views"], sum(w * h for w, h in [S.BATCH_RESOLUTIONS[k // 2] for k in range(case["views"])])
    else:
        views = case["views"] if kind == "autograd" else 1
        px = views * case["width"] * case["height"]
    forward = views * n * (250 + 2 * (f - 11)) + px * (60 * 27 + 3 * 5 * 44)
    backward = views * n * (600 + 6 * (f - 11)) + px * (60 * 62 + 3 * 3 * 44)
    images = 2 * 12 * px
    return {
        "step": dict(bytes=24 * f * n + images, flops=forward + backward + 12 * f * n),
        "grow": dict(bytes=24 * f * n + images + 16 * n, flops=forward + backward + 12 * f * n),
        "batch": dict(bytes=24 * f * n + images, flops=forward + backward + 12 * f * n),
        "skip": dict(bytes=4 * f * n + images, flops=forward),
        "eval": dict(bytes=4 * f * n + images, flops=forward),
        "autograd": dict(bytes=8 * f * n + images, flops=forward + backward),
        "loss": dict(bytes=36 * px, flops=px * 3 * 8 * 44),
        "densify": dict(bytes=12 * f * n + 32 * n + 13 * f * n, flops=20 * n),
    }[kind]


# ---------------------------------------------------------------------------
# The same results in 64 bits, in plain torch
# ---------------------------------------------------------------------------
def _loss64(x, y, w, h):
    x, y = x.reshape(1, 3, h, w), y.reshape(1, 3, h, w)
    k = torch.exp(-(torch.arange(11, dtype=torch.float64, device=x.device) - 5) ** 2 / (2 * 1.5 ** 2))
    k = k / k.sum()

    def window(a):
        a = torch.nn.functional.pad(a, (5, 5, 5, 5))
        a = sum(k[i] * a[..., :, i:i + w] for i in range(11))
        return sum(k[i] * a[..., i:i + h, :] for i in range(11))

    mx, my = window(x), window(y)
    sxx, syy, sxy = window(x * x) - mx * mx, window(y * y) - my * my, window(x * y) - mx * my
    c1, c2 = 0.01 ** 2, 0.03 ** 2
    ssim = (2 * mx * my + c1) * (2 * sxy + c2) / ((mx * mx + my * my + c1) * (sxx + syy + c2))
    return (1 - LAM) * (x - y).abs().mean() + LAM * (1 - ssim.mean())


def _sh64(d, degree):
    """Real spherical harmonics with the Condon-Shortley phase at unit directions d [n, 3]."""
    x, y, z = d.unbind(1)
    c = [math.sqrt(1 / (4 * math.pi)), math.sqrt(3 / (4 * math.pi)), math.sqrt(15 / (4 * math.pi)),
         math.sqrt(5 / (16 * math.pi)), math.sqrt(35 / (32 * math.pi)), math.sqrt(105 / (4 * math.pi)),
         math.sqrt(21 / (32 * math.pi)), math.sqrt(7 / (16 * math.pi))]
    out = [torch.full_like(x, c[0])]
    if degree > 0:
        out += [-c[1] * y, c[1] * z, -c[1] * x]
    if degree > 1:
        out += [c[2] * x * y, -c[2] * y * z, c[3] * (3 * z * z - 1), -c[2] * x * z, c[2] / 2 * (x * x - y * y)]
    if degree > 2:
        out += [-c[4] * y * (3 * x * x - y * y), c[5] * x * y * z, -c[6] * y * (5 * z * z - 1),
                c[7] * z * (5 * z * z - 3), -c[6] * x * (5 * z * z - 1), c[5] / 2 * z * (x * x - y * y),
                -c[4] * x * (x * x - 3 * y * y)]
    return torch.stack(out, 1)


def _render64(p, n, sh, cam):
    """Image [3, H, W] of one view of the planes p [F, n] (binary64): every Gaussian at every pixel."""
    rp, dev = sk.RasterParams(), p.device
    f32 = lambda v: float(np.float32(v))  # noqa: E731
    R = torch.as_tensor(np.asarray(cam.R, np.float64), device=dev)
    t = torch.as_tensor(np.asarray(cam.t, np.float64), device=dev)
    mu = p[0:3].T
    tc = mu @ R.T + t
    near = tc[:, 2].detach() > f32(rp.near_z)
    mu, tc, p = mu[near], tc[near], p[:, near]
    q = p[6:10] / p[6:10].norm(dim=0, keepdim=True)
    w, x, y, z = q
    rot = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                       2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                       2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1).reshape(-1, 3, 3)
    M = rot * p[3:6].T.exp()[:, None, :]
    tx, ty, tz = tc.unbind(1)
    lx, ly = (f32(rp.jac_clamp) * (a / 2) / b for a, b in ((cam.width, cam.fx), (cam.height, cam.fy)))
    xr, yr, o = (tx / tz).clamp(-lx, lx), (ty / tz).clamp(-ly, ly), torch.zeros_like(tz)
    J = torch.stack([cam.fx / tz, o, -cam.fx * xr / tz, o, cam.fy / tz, -cam.fy * yr / tz], 1).reshape(-1, 2, 3)
    A = J @ R @ M
    cov = A @ A.transpose(1, 2)
    sxx, sxy, syy = cov[:, 0, 0] + f32(rp.dilation), cov[:, 0, 1], cov[:, 1, 1] + f32(rp.dilation)
    det = sxx * syy - sxy * sxy
    u, v = cam.fx * tx / tz + cam.cx, cam.fy * ty / tz + cam.cy
    opa = torch.sigmoid(p[10])
    d = mu - (-(R.T @ t))
    Y = _sh64(d / d.norm(dim=1, keepdim=True), sh)
    rgb = ((Y[:, :, None] * p[11:].T.reshape(len(Y), -1, 3)).sum(1) + 0.5).clamp(min=0)
    with torch.no_grad():
        mid = 0.5 * (sxx + syy)
        r = torch.ceil(3 * (mid + (mid * mid - det).clamp(min=0).sqrt()).sqrt())
        tau = torch.log(opa / f32(rp.alpha_min))
        rx, ry = (torch.minimum(r, torch.ceil((2 * tau.clamp(min=0) * s).sqrt())) for s in (sxx, syy))
        order = torch.sort(tc[:, 2].float(), stable=True)[1]
    u, v, sxx, sxy, syy, det, opa, rgb, rx, ry, tau = (
        a[order] for a in (u, v, sxx, sxy, syy, det, opa, rgb, rx, ry, tau))
    px = torch.arange(cam.width, device=dev, dtype=torch.float64) + 0.5
    py = torch.arange(cam.height, device=dev, dtype=torch.float64) + 0.5
    dx, dy = px[None, None, :] - u[:, None, None], py[None, :, None] - v[:, None, None]
    s = lambda a: (a / det)[:, None, None]  # noqa: E731
    power = -0.5 * (s(syy) * dx * dx + s(sxx) * dy * dy) + s(sxy) * dx * dy
    raw = opa[:, None, None] * power.exp()
    with torch.no_grad():
        take = (dx.abs() <= rx[:, None, None]) & (dy.abs() <= ry[:, None, None]) & (tau >= 0)[:, None, None]
        take &= (power <= 0) & (raw >= f32(rp.alpha_min))
    alpha = torch.where(take, raw.clamp(max=f32(rp.alpha_max)), torch.zeros_like(raw))
    with torch.no_grad():  # a pixel stops before the Gaussian that would take it below t_min
        go = (torch.cumprod(1 - alpha, 0) >= f32(rp.t_min)).double()
    alpha = alpha * go
    left = torch.cumprod(1 - alpha, 0)
    before = torch.cat([torch.ones_like(left[:1]), left[:-1]])
    return ((alpha * before)[:, None] * rgb[:, :, None, None]).sum(0)


def exact(case, seed):
    kind, n = case["kind"], case["n"]
    if kind == "loss":
        rgb, target = _images(case, seed)
        x = rgb.double().requires_grad_(True)
        loss = _loss64(x, target.double(), case["width"], case["height"])
        loss.backward()
        return dict(loss=loss.detach().reshape(1), dl=x.grad)
    if kind == "autograd" and n * case["width"] * case["height"] <= 8_000_000:
        s = prepare(case, seed)
        x, loss, at, images = s["planes"].detach()[:, :n].double().requires_grad_(True), 0.0, 0, []
        for c, px in zip(s["cams"], s["px"]):
            img = _render64(x, n, case["sh"], c)
            loss = loss + _loss64(img, s["target"][at:at + 3 * px].double(), c.width, c.height)
            images.append(img.detach().reshape(-1))
            at += 3 * px
        loss.backward()
        grad = torch.zeros(s["planes"].shape, dtype=torch.float64, device="cuda")
        grad[:, :n] = x.grad
        return dict(rgb=torch.cat(images), loss=loss.detach(), grad=grad)
    if kind == "densify":
        p, planes, m, v, grad_sum, count, normals = _densify_inputs(case, seed)
        a = planes[:, :n]
        alive = a[10] >= float(np.float32(math.log(p.min_opacity / (1 - p.min_opacity))))
        grow = (count > 0) & (grad_sum.double() >= float(np.float32(p.grad_threshold)) * count.double()) & alive
        large = a[3:6].amax(0) > float(np.float32(math.log(np.float32(p.percent_dense) * float(np.float32(p.scene_extent)))))
        keep, clone, split = (torch.nonzero(k).flatten() for k in (alive & ~(grow & large), grow & ~large, grow & large))
        w, x, y, z = a[6:10, split].double() / a[6:10, split].double().norm(dim=0, keepdim=True)
        rot = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                           2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                           2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1).reshape(-1, 3, 3)
        step = (normals[split].double() * a[3:6, split].T.double().exp()[:, None, :]) @ rot.transpose(1, 2)
        child = a[:, split].double()[:, :, None].repeat(1, 1, 2)
        child[0:3] += step.permute(2, 0, 1)
        child[3:6] -= math.log(float(np.float32(p.split_scale)))
        first, after = len(keep) + len(clone), len(keep) + len(clone) + 2 * len(split)
        out = [torch.zeros(planes.shape[0], S.padded_stride(2 * n), dtype=torch.float64, device="cuda") for _ in range(3)]
        out[0][:, :len(keep)], out[0][:, len(keep):first] = a[:, keep], a[:, clone]
        out[0][:, first:after] = child.reshape(planes.shape[0], -1)
        out[1][:, :len(keep)], out[2][:, :len(keep)] = m[:, keep], v[:, keep]
        return dict(planes=out[0], m=out[1], v=out[2], n=torch.tensor([after], device="cuda"))
    return None
