"""Workloads the rasterizer is timed on, with an independent FP64 value of each.

`listed()` are fixed cases, `draw(rng)` makes further ones of the same ranges.
A case names an entry point, a particle set and cameras:

  entry     "project" (gut_project alone), "forward" (project -> bin -> render),
            "train" (render_gaussians and its gradients), "serve" (requests to
            the continuous-batching server)
  n, sh     particles and SH degree; layout "uniform" (a unit box of blobs) or
            "clustered" (200 anisotropic clusters plus a distant shell)
  cams      cameras per call (per request when serving); model "pinhole",
            "fisheye" (OpenCV, 180 degrees) or "both" in turn; rolling shutter
  degree    degree of the response (2: Gaussian); kbuffer: the per-ray buffer's
            size (0: tile order); clip: a per-pixel clip distance

`prepare` draws everything on the GPU from the seed; `exact` evaluates the
method densely in FP64 with plain torch.
"""
import math

import numpy as np
import torch

from paper_2412_12507_amd import raster as R
from paper_2412_12507_amd.serve import Server

ALPHA_MIN, ALPHA_MAX, T_MIN, NEAR, K_MAX, TILE = 1.0 / 255.0, 0.99, 1e-4, 0.2, 3.0, 16
SH_C0 = 0.5 / math.sqrt(math.pi)
PAN, SHIFT = 0.1, 0.3  # rolling shutter: radians about the camera's y, units along its x


def _case(name, entry, n, width, height, *, layout="clustered", sh=3, cams=1, model="pinhole",
          rolling=False, degree=2, kbuffer=0, clip=False, requests=0):
    c = dict(entry=entry, n=n, layout=layout, sh=sh, width=width, height=height, cams=cams,
             model=model, rolling=rolling, degree=degree, kbuffer=kbuffer, clip=clip,
             requests=requests)
    return dict(c, name=name) if name else c


def listed():
    return [
        # a thumbnail of a toy scene: launches and host work are all there is
        _case("forward_1k_128", "forward", 1_000, 128, 128, layout="uniform", sh=0),
        # a preview of a small scene at an odd size, with a wide lens
        _case("forward_30k_fisheye_517x291", "forward", 30_000, 517, 291, model="fisheye", sh=2),
        # projection alone, as a caller with its own binning uses it: two views share the scene's read
        _case("project_1m_two_1080p", "project", 1_000_000, 1920, 1080, cams=2, model="both"),
        # the headline: a trained scene's size, two Full-HD views in one call
        _case("forward_1m_two_1080p", "forward", 1_000_000, 1920, 1080, cams=2, model="both"),
        # a driving scene's size under a rolling shutter
        _case("forward_3m_rolling_1600x1200", "forward", 3_000_000, 1600, 1200, model="fisheye",
              rolling=True),
        # rasterized primary rays of a hybrid renderer: degree-4 response, clip distance per pixel
        _case("hybrid_1m_1280x720", "forward", 1_000_000, 1280, 720, degree=4, clip=True),
        # a fitting step on a small scene, odd sizes, lower SH degree
        _case("train_5k_250x187", "train", 5_000, 250, 187, layout="uniform", sh=1),
        # a training step of a full scene: one Full-HD view forward and backward
        _case("train_1m_fisheye_1080p", "train", 1_000_000, 1920, 1080, model="fisheye"),
        # a training step on a rolling-shutter capture
        _case("train_300k_rolling_800x600", "train", 300_000, 800, 600, model="fisheye", rolling=True),
        # the sorted variant (k = 16): quality renders, two views
        _case("sorted_1m_two_1080p", "forward", 1_000_000, 1920, 1080, cams=2, model="both", kbuffer=16),
        # a training step of the sorted variant
        _case("sorted_train_300k_1280x720", "train", 300_000, 1280, 720, model="fisheye", kbuffer=16),
        # a resident scene serving a burst of three requests of two mixed cameras
        _case("serve_3m_three_requests", "serve", 3_000_000, 1920, 1080, cams=2, model="both", requests=3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    entry = rng.choice(["project", "forward", "forward", "forward", "train", "train", "train", "serve"])
    n = _log(rng, 1_000, 2_000_000) if entry != "serve" else _log(rng, 200_000, 2_000_000)
    width = _log(rng, 120, 1920)
    height = max(90, int(width * rng.uniform(0.5, 0.85)))
    model = rng.choice(["pinhole", "fisheye", "both"])
    kbuffer = rng.choice([0, 0, 16, rng.randint(1, 16)]) if entry in ("forward", "train") else 0
    return _case(None, entry, n, width, height, layout="uniform" if n < 10_000 else "clustered",
                 sh=rng.choice([0, 1, 2, 3, 3, 3]), cams=rng.choice([1, 1, 2]) if entry != "train" else 1,
                 model=model, rolling=rng.random() < 0.3,
                 degree=rng.choice([2, 2, 2, 3, 4, 8]) if entry != "project" else 2,
                 kbuffer=kbuffer, clip=entry in ("forward", "train") and rng.random() < 0.2,
                 requests=rng.randint(1, 4) if entry == "serve" else 0)


# ---------------------------------------------------------------------- inputs

def _unit(v):
    return v / np.linalg.norm(v)


def _camera(case, fisheye, rng, rolling):
    """A camera dict at radius 8 (clustered) or 3 (uniform) looking at the origin."""
    while True:
        eye = _unit(rng.normal(size=3))
        if abs(eye[1]) < 0.95:
            break
    eye *= 8.0 if case["layout"] == "clustered" else 3.0
    z = _unit(-eye)
    x = _unit(np.cross([0.0, 1.0, 0.0], z))
    R0 = np.stack([x, np.cross(z, x), z])
    w, h = case["width"], case["height"]
    if fisheye:
        f, k = (w / 2.0) / (math.pi / 2.0), [float(v) for v in rng.uniform(-0.05, 0.05, 4)]
    else:
        f, k = (w / (2.0 * math.tan(math.pi / 6.0)) if case["layout"] == "clustered" else 150.0 * w / 128.0), [0.0] * 4
    R1, c1 = R0, eye
    if rolling:
        s, c = math.sin(PAN), math.cos(PAN)
        R1 = (R0.T @ np.array([[c, 0.0, s], [0.0, 1.0, 0.0], [-s, 0.0, c]])).T
        c1 = eye + SHIFT * x
    return dict(model="fisheye" if fisheye else "pinhole", shutter="rolling" if rolling else "global",
                width=w, height=h, fx=f, fy=f, cx=w / 2.0, cy=h / 2.0, k=k,
                R0=R0, t0=-R0 @ eye, R1=R1, t1=-R1 @ c1)


def _cameras(case, seed):
    """The cameras of one call, or of each request in turn."""
    rng = np.random.default_rng(2000 + seed)
    out = []
    for i in range(case["cams"] * max(1, case["requests"])):
        fisheye = case["model"] == "fisheye" or (case["model"] == "both" and i % 2 == 1)
        # a served camera pair mixes a still lens with a rolling-shutter one
        out.append(_camera(case, fisheye, rng, case["rolling"] or (case["entry"] == "serve" and fisheye)))
    return out


def _scene(case, seed):
    """Activated particle parameters (float32 on the GPU)."""
    dev = torch.device("cuda")
    g = torch.Generator(device=dev).manual_seed(1000 + seed)
    nrm = lambda *s: torch.randn(*s, generator=g, device=dev)
    uni = lambda *s: torch.rand(*s, generator=g, device=dev)
    n, K = case["n"], (case["sh"] + 1) ** 2
    if case["layout"] == "uniform":
        means, log_s = uni(n, 3) * 2 - 1, -3.5 + 0.5 * nrm(n, 3)
    else:
        m = n - n // 5
        owner = torch.arange(m, device=dev) * 200 // m  # clusters are runs of neighbouring ids
        centre, axes = uni(200, 3) * 10 - 5, 0.3 * (0.5 + uni(200, 3))
        rot = torch.linalg.qr(nrm(200, 3, 3).cpu())[0].to(dev)
        clu = centre[owner] + ((nrm(m, 3) * axes[owner])[:, None, :] * rot[owner]).sum(2)
        far = nrm(n - m, 3)
        means = torch.cat([clu, 20 * far / far.norm(dim=1, keepdim=True)])
        log_s = -4.0 + 0.7 * nrm(n, 3)
    quats = nrm(n, 4)
    sh = 0.05 * nrm(n, K, 3)
    sh[:, 0] = (uni(n, 3) - 0.5) / SH_C0
    return R.GaussianScene(means.contiguous(), log_s.exp(), quats / quats.norm(dim=1, keepdim=True),
                           torch.sigmoid(nrm(n)), sh, case["sh"])


def _per_pixel(case, seed):
    """The clip distances, and the loss gradients a training step starts from (an L1 loss's +-1/N)."""
    g = torch.Generator(device="cuda").manual_seed(3000 + seed)
    px = case["width"] * case["height"] * case["cams"]
    lo, hi = (6.0, 10.0) if case["layout"] == "clustered" else (2.5, 4.0)
    clip = lo + (hi - lo) * torch.rand(px, generator=g, device="cuda") if case["clip"] else None
    d_rgb = None
    if case["entry"] == "train":
        d_rgb = torch.sign(torch.rand(case["height"], case["width"], 3, generator=g, device="cuda") - 0.5) / (3 * px)
    return clip, d_rgb


def _params(case):
    return dict(kernel_degree=case["degree"], kbuffer=case["kbuffer"])


def prepare(case, seed):
    scene, cams = _scene(case, seed), _cameras(case, seed)
    s = dict(case=case, scene=scene, cams=cams, params=_params(case))
    s["clip"], s["d_rgb"] = _per_pixel(case, seed)
    if case["entry"] == "train":
        s["leaves"] = [t.requires_grad_(True) for t in
                       (scene.means, scene.scales, scene.quats, scene.opacities, scene.sh)]
    elif case["entry"] == "serve":
        k = case["cams"]
        s["requests"] = [cams[i:i + k] for i in range(0, len(cams), k)]
        s["server"] = Server(scene, s["params"], mem_budget_bytes=24 << 30, max_slots=4, max_batch_cams=8)
    return s


def run(s):
    case, cams = s["case"], s["cams"]
    if case["entry"] == "project":
        p = R.project(s["scene"], cams, s["params"])
        return dict(rect=p.rect, tiles=p.tiles, depth=p.depth, rgb=p.rgb, record=p.record,
                    mean2d=p.mean2d, extent=p.extent)
    if case["entry"] == "forward":
        _, _, img = R.forward(s["scene"], cams, s["params"], clip=s["clip"])
        return dict(rgb=img.rgb, T=img.T, n_contrib=img.n_contrib)
    if case["entry"] == "train":
        imgs, Ts = R.render_gaussians(*s["leaves"], case["sh"], cams, s["params"], clip=s["clip"])
        g = torch.autograd.grad(imgs, s["leaves"], [s["d_rgb"]])
        return dict(image=imgs[0], T=Ts[0], means=g[0], scales=g[1], quats=g[2], opacities=g[3], sh=g[4])
    srv = s["server"]
    ids = [srv.submit(r)[0] for r in s["requests"]]
    return dict(images=[srv.wait(i) for i in ids])


def work(case):
    """What the method must move and compute: the particles once, each camera's pixels once; about
    600 FLOPs per (camera, particle) projected and, for each pixel, some 40 blended hits at 55 FLOPs
    (the response, Eq. 11, and the blend), three times that with the backward."""
    K, n = (case["sh"] + 1) ** 2, case["n"]
    cams = case["cams"] * max(1, case["requests"])
    px = case["width"] * case["height"] * cams
    particle = 4 * (11 + 3 * K)
    if case["entry"] == "project":
        return dict(bytes=n * particle + n * 64 + n * cams * 52, flops=600 * n * cams)
    if case["entry"] == "train":
        return dict(bytes=3 * n * particle + px * (16 + 12 + 4), flops=1200 * n + px * 3 * 40 * 55)
    out = 12 if case["entry"] == "serve" else 20
    return dict(bytes=n * particle + px * (out + (4 if case["clip"] else 0)), flops=600 * n * cams + px * 40 * 55)


# ------------------------------------------------------------ the same in FP64

def _rotation(q):
    w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                        2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                        2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1).view(-1, 3, 3)


def _apply(M, v):
    """M [.., 3, 3] times v [.., 3], without a batched product."""
    return (M * v[..., None, :]).sum(-1)


def _sh_basis(d, degree):
    x, y, z = d.unbind(1)
    s = lambda num: math.sqrt(num / math.pi)
    Y = [0 * x + SH_C0]
    if degree >= 1:
        Y += [-s(0.75) * y, s(0.75) * z, -s(0.75) * x]
    if degree >= 2:
        Y += [s(3.75) * x * y, -s(3.75) * y * z, s(5 / 16) * (2 * z * z - x * x - y * y),
              -s(3.75) * x * z, s(15 / 16) * (x * x - y * y)]
    if degree >= 3:
        a, b, c, d7, e = s(35 / 32), s(105 / 4), s(21 / 32), s(7 / 16), s(105 / 16)
        Y += [-a * y * (3 * x * x - y * y), b * x * y * z, -c * y * (4 * z * z - x * x - y * y),
              d7 * z * (2 * z * z - 3 * x * x - 3 * y * y), -c * x * (4 * z * z - x * x - y * y),
              e * z * (x * x - y * y), -a * x * (x * x - 3 * y * y)]
    return torch.stack(Y, 1)


class _Cam64:
    """A camera in FP64: pose over the exposure, projection and pixel rays."""

    def __init__(self, cam, dev):
        t = lambda a: torch.as_tensor(np.asarray(a, np.float64), device=dev)
        self.fish, self.rolling = cam["model"] == "fisheye", cam["shutter"] == "rolling"
        self.W, self.H = cam["width"], cam["height"]
        self.fx, self.fy, self.cx, self.cy, self.k = cam["fx"], cam["fy"], cam["cx"], cam["cy"], cam["k"]
        self.R0 = t(cam["R0"])
        self.c0 = t(-np.asarray(cam["R0"]).T @ cam["t0"])
        self.dc = t(-np.asarray(cam["R1"]).T @ cam["t1"]) - self.c0
        self.tx, self.ty = -(-self.W // TILE), -(-self.H // TILE)
        th = np.linspace(0.0, math.pi / 2, 200001)
        down = np.nonzero(self._slope(th) <= 0)[0]
        self.lim = math.pi / 2
        if self.fish and len(down):
            lo, hi = th[down[0] - 1], th[down[0]]
            for _ in range(80):
                mid = 0.5 * (lo + hi)
                lo, hi = (mid, hi) if self._slope(mid) > 0 else (lo, mid)
            self.lim = lo

    def _slope(self, th):
        return 1 + sum((2 * i + 3) * k * th ** (2 * i + 2) for i, k in enumerate(self.k))

    def _theta_d(self, th):
        return th * (1 + sum(k * th ** (2 * i + 2) for i, k in enumerate(self.k)))

    def _pan(self, y, t, sign):
        """y turned by sign * t * PAN about the camera's y axis."""
        if not self.rolling:
            return y
        s, c = torch.sin(t * PAN) * sign, torch.cos(t * PAN)
        return torch.stack([c * y[..., 0] + s * y[..., 2], y[..., 1], c * y[..., 2] - s * y[..., 0]], -1)

    def centre(self, t):
        return self.c0 + t[..., None] * self.dc if self.rolling else self.c0.expand(*t.shape, 3)

    def project_at(self, x, t):
        p = self._pan(_apply(self.R0, x - self.centre(t)), t, -1.0)
        if not self.fish:
            return self.fx * p[:, 0] / p[:, 2] + self.cx, self.fy * p[:, 1] / p[:, 2] + self.cy, p[:, 2] > NEAR
        r = torch.hypot(p[:, 0], p[:, 1])
        th = torch.atan2(r, p[:, 2])
        sc = self._theta_d(th) / r.clamp_min(1e-300)
        return (self.fx * sc * p[:, 0] + self.cx, self.fy * sc * p[:, 1] + self.cy,
                (th <= self.lim) & (p.norm(dim=1) > NEAR))

    def project(self, x):
        """(u, v, valid, exposure time), the time by three row iterations."""
        t = torch.zeros_like(x[:, 0])
        if self.rolling:
            t = t + 0.5
            for _ in range(3):
                _, v, ok = self.project_at(x, t)
                t = torch.where(ok, ((v - 0.5) / (self.H - 1)).clamp(0, 1), t)
        return (*self.project_at(x, t), t)

    def rays(self, px, py):
        """World ray (origin, direction, valid) of pixels."""
        t = py.double() / (self.H - 1) if self.rolling else torch.zeros(px.shape, dtype=torch.float64, device=px.device)
        x, y = (px.double() + 0.5 - self.cx) / self.fx, (py.double() + 0.5 - self.cy) / self.fy
        if not self.fish:
            d, ok = torch.stack([x, y, torch.ones_like(x)], -1), torch.ones_like(x, dtype=torch.bool)
        else:
            td = torch.hypot(x, y)
            ok = td <= self._theta_d(self.lim)
            lo, hi = torch.zeros_like(td), torch.full_like(td, self.lim)
            for _ in range(60):
                mid = 0.5 * (lo + hi)
                up = self._theta_d(mid) < td
                lo, hi = torch.where(up, mid, lo), torch.where(up, hi, mid)
            sc = torch.sin(hi) / td.clamp_min(1e-300)
            d = torch.stack([sc * x, sc * y, torch.cos(hi)], -1)
        return self.centre(t), _apply(self.R0.T, self._pan(d, t, 1.0)), ok


def _exact_project(S, cam, case):
    """UT projection of every particle (alpha = 1, beta = 2, kappa = 0: lambda = 0)."""
    mu, s, sig = S["means"], S["scales"], S["opacities"]
    Rm = _rotation(S["quats"])
    pts = [mu] + [mu + sg * math.sqrt(3.0) * s[:, k:k + 1] * Rm[:, :, k] for sg in (1, -1) for k in range(3)]
    u, v, ok, t = zip(*(cam.project(p) for p in pts))
    u, v, ok, t0 = torch.stack(u, 1), torch.stack(v, 1), torch.stack(ok, 1).all(1), t[0]
    mean = torch.stack([u[:, 1:].mean(1), v[:, 1:].mean(1)], 1)
    du, dv = u - mean[:, :1], v - mean[:, 1:]
    w = torch.tensor([2.0] + [1 / 6] * 6, dtype=torch.float64, device=mu.device)
    cov = torch.stack([(w * du * du).sum(1), (w * du * dv).sum(1), (w * dv * dv).sum(1)], 1)
    deg = case["degree"]
    lam = 0.5 * 3.0 ** (2 - deg)
    k = ((sig / ALPHA_MIN).log().clamp_min(0) / lam).pow(1.0 / deg).clamp_max(K_MAX)
    h = k[:, None] * torch.stack([cov[:, 0], cov[:, 2]], 1).clamp_min(0).sqrt()
    big = torch.tensor([cam.tx, cam.ty], dtype=torch.float64, device=mu.device)
    lo = torch.minimum(((mean - h) / TILE).floor().clamp_min(0), big)
    hi = torch.maximum(torch.minimum(((mean + h) / TILE).floor(), big - 1), lo * 0 - 1)
    vis = ok & (sig >= ALPHA_MIN) & (lo <= hi).all(1)
    dv3 = mu - cam.centre(t0)
    dist = dv3.norm(dim=1)
    return dict(mean=mean, A=k[:, None] ** 2 * cov, k=k, lo=lo.nan_to_num().long(), hi=hi.nan_to_num().long(),
                vis=vis, depth=dist, t0=t0)


def _exact_rgb(mu, sh, centre, degree):
    d = mu - centre
    Y = _sh_basis(d / d.norm(dim=1, keepdim=True), degree)
    return (0.5 + (Y[:, :, None] * sh).sum(1)).clamp_min(0)


def _exact_lists(P, cam):
    """(tile, particle) pairs whose extent ellipse meets the tile's box, in (tile, depth, id) order."""
    idx = P["vis"].nonzero()[:, 0]
    lo, hi = P["lo"][idx], P["hi"][idx]
    nx, area = hi[:, 0] - lo[:, 0] + 1, (hi - lo + 1).prod(1)
    own = torch.repeat_interleave(torch.arange(len(idx), device=idx.device), area)
    r = torch.arange(len(own), device=idx.device) - (area.cumsum(0) - area)[own]
    tx, ty, e = lo[own, 0] + r % nx[own], lo[own, 1] + r // nx[own], idx[own]
    a, b, c = P["A"][e].unbind(1)
    det = a * c - b * b
    N11, N12, N22 = c / det, -b / det, a / det
    x0, y0 = tx * float(TILE) - P["mean"][e, 0], ty * float(TILE) - P["mean"][e, 1]
    x1, y1 = x0 + TILE, y0 + TILE

    def edge(x, l, h, nxx, nyy):
        y = torch.minimum(torch.maximum(-N12 * x / nyy, l), h)
        return nxx * x * x + 2 * N12 * x * y + nyy * y * y <= 1

    keep = (x0 <= 0) & (x1 >= 0) & (y0 <= 0) & (y1 >= 0)
    keep |= edge(x0, y0, y1, N11, N22) | edge(x1, y0, y1, N11, N22)
    keep |= edge(y0, x0, x1, N22, N11) | edge(y1, x0, x1, N22, N11)
    keep |= ~(det > 0)
    tile, e = (ty * cam.tx + tx)[keep], e[keep]
    rank = torch.empty_like(P["depth"], dtype=torch.int64)
    rank[torch.argsort(P["depth"], stable=True)] = torch.arange(len(rank), device=rank.device)
    e = e[torch.argsort(tile * len(rank) + rank[e])]
    return e, torch.bincount(tile, minlength=cam.tx * cam.ty)


def _alpha(mu, M, sig, o, d, case):
    """alpha (0 where nothing is hit) and the hit's distance, over broadcast pixels and particles."""
    og, dg = _apply(M, o - mu), _apply(M, d)
    cr = torch.linalg.cross(og, dg)
    dd, od = (dg * dg).sum(-1), (og * dg).sum(-1)
    w2 = (cr * cr).sum(-1) / dd
    deg = case["degree"]
    lam = 0.5 * 3.0 ** (2 - deg)
    a = sig * torch.exp(-lam * (w2 if deg == 2 else w2 ** (0.5 * deg)))
    hit = (od < 0) & (a >= ALPHA_MIN)
    return torch.where(hit, a.clamp_max(ALPHA_MAX), torch.zeros_like(a)), (-od / dd).detach() * d.norm(dim=-1)


def _groups(count, most):
    """Tiles of similar list length, longest first, each group padded to about `most` evaluations."""
    order = torch.argsort(count, descending=True)
    n, i = count[order].cpu().tolist(), 0
    while i < len(n) and n[i] > 0:
        g = max(1, most // (n[i] * TILE * TILE))
        j = i
        while j < len(n) and j < i + g and n[j] > 0:
            j += 1
        yield order[i:j], n[i]
        i = j


def _tile_rays(cam, tiles, clip):
    q = torch.arange(TILE * TILE, device=tiles.device)
    px = (tiles % cam.tx)[:, None] * TILE + q % TILE
    py = (tiles // cam.tx)[:, None] * TILE + q // TILE
    o, d, ok = cam.rays(px, py)
    inside = (px < cam.W) & (py < cam.H)
    pix = torch.where(inside, py * cam.W + px, torch.zeros_like(px))
    return o, d, ok & inside, inside, pix, None if clip is None else clip[pix].double()


def _exact_sorted(a, dist, col, k):
    """Multi-layer alpha blending with a buffer of the k farthest hits; a, dist [.., L]."""
    T, done = torch.ones_like(a[..., 0]), torch.zeros_like(a[..., 0], dtype=torch.bool)
    C = torch.zeros(*T.shape, 3, dtype=T.dtype, device=T.device)
    bd = torch.full((*T.shape, k), -math.inf, dtype=T.dtype, device=T.device)
    ba, bi = torch.zeros_like(bd), torch.zeros_like(bd, dtype=torch.int64)

    def blend(al, i):
        nonlocal T, done, C
        Tn = T * (1 - al)
        go = (al > 0) & ~done
        done = done | (go & (Tn < T_MIN))
        go = go & ~done
        rgb = torch.gather(col, 1, i[..., None].expand(*i.shape, 3))
        C = C + torch.where(go, al * T, torch.zeros_like(T))[..., None] * rgb
        T = torch.where(go, Tn, T)

    for j in range(a.shape[-1]):
        aj, dj = a[..., j], dist[..., j]
        hit = (aj > 0) & ~done
        if not bool(hit.any()):
            continue
        near, slot = bd.min(-1)
        ij = torch.full_like(slot, j)
        evict = hit & (dj > near)
        one = slot[..., None]
        blend(torch.where(hit, torch.where(evict, ba.gather(-1, one)[..., 0], aj), torch.zeros_like(aj)),
              torch.where(evict, bi.gather(-1, one)[..., 0], ij))
        for buf, new in ((bd, dj), (ba, aj), (bi, ij)):
            buf.scatter_(-1, one, torch.where(evict, new, buf.gather(-1, one)[..., 0])[..., None])
    bd, at = bd.sort(-1)
    for j in range(k):
        blend(ba.gather(-1, at)[..., j], bi.gather(-1, at)[..., j])
    return C, T


def _exact_image(S, cam, case, clip, d_rgb=None, grads=None):
    """(rgb [P,3], T [P]); with d_rgb adds dL/d(means, M, opacities, rgb) to grads."""
    P = _exact_project(S, cam, case)
    e, count = _exact_lists(P, cam)
    start = count.cumsum(0) - count
    npx = cam.W * cam.H
    out, out_T = torch.zeros(npx, 3, dtype=torch.float64, device=e.device), torch.ones(npx, dtype=torch.float64, device=e.device)
    M = _rotation(S["quats"]).transpose(1, 2) / S["scales"][:, :, None]
    rgb = _exact_rgb(S["means"], S["sh"], cam.centre(P["t0"]), case["sh"])
    for tiles, L in _groups(count, 1 << 22 if d_rgb is None else 1 << 21):
        o, d, ok, inside, pix, cl = _tile_rays(cam, tiles, clip)
        at = start[tiles][:, None] + torch.arange(L, device=e.device)
        real = torch.arange(L, device=e.device) < count[tiles][:, None]
        i = e[torch.where(real, at, torch.zeros_like(at))]
        part = [S["means"][i], M[i], S["opacities"][i], rgb[i]]
        if d_rgb is not None:
            part = [t.detach().requires_grad_(True) for t in part]
        with torch.set_grad_enabled(d_rgb is not None):
            a, dist = _alpha(part[0][:, None], part[1][:, None], part[2][:, None], o[:, :, None], d[:, :, None], case)
            drop = ~(real[:, None] & ok[:, :, None])
            if cl is not None:
                drop |= dist > cl[:, :, None]
            a = torch.where(drop, torch.zeros_like(a), a)
            if case["kbuffer"]:
                C, T = _exact_sorted(a, dist, part[3], case["kbuffer"])
            else:
                # once the running product is below T_MIN, neither this hit nor a later one is added
                a = torch.where(torch.cumprod(1 - a.detach(), 2) < T_MIN, torch.zeros_like(a), a)
                inc = torch.cumprod(1 - a, 2)
                T = inc[:, :, -1]
                before = torch.cat([torch.ones_like(inc[:, :, :1]), inc[:, :, :-1]], 2)
                C = ((a * before)[..., None] * part[3][:, None]).sum(2)
            if d_rgb is not None:
                g = torch.autograd.grad((C * d_rgb[pix] * inside[..., None]).sum(), part)
                for acc, x in zip(grads, g):
                    acc.index_add_(0, i.reshape(-1), (x * real.view(*real.shape, *[1] * (x.dim() - 2))).flatten(0, 1))
        out[pix[inside]], out_T[pix[inside]] = C.detach()[inside], T.detach()[inside]
    return out, out_T


def exact(case, seed):
    s, cams = _scene(case, seed), _cameras(case, seed)
    clip, d_rgb = _per_pixel(case, seed)
    S = {k: getattr(s, k).double() for k in ("means", "scales", "quats", "opacities", "sh")}
    dev = S["means"].device
    c64 = [_Cam64(c, dev) for c in cams]
    M = _rotation(S["quats"]).transpose(1, 2) / S["scales"][:, :, None]
    if case["entry"] == "project":
        depth, rgb, extent = [], [], []
        for cam in c64:
            P = _exact_project(S, cam, case)
            zero = lambda x: torch.where(P["vis"].view(-1, *[1] * (x.dim() - 1)), x, torch.zeros_like(x))
            depth.append(zero(P["depth"]))
            rgb.append(zero(_exact_rgb(S["means"], S["sh"], cam.centre(P["t0"]), case["sh"])))
            extent.append(zero(torch.cat([P["A"], P["k"][:, None]], 1)))
        record = torch.zeros(case["n"], 16, dtype=torch.float64, device=dev)
        record[:, :3], record[:, 3] = S["means"], S["opacities"]
        record.view(-1, 4, 4)[:, 1:, :3] = M
        # (a culled entry's mean is whatever its invalid points gave)
        return dict(rect=None, tiles=None, depth=torch.cat(depth), rgb=torch.cat(rgb), record=record,
                    mean2d=None, extent=torch.cat(extent))
    px = case["width"] * case["height"]
    if case["entry"] == "train":
        sorted_ = case["kbuffer"] > 0
        grads = [torch.zeros_like(x) for x in (S["means"], M, S["opacities"], S["means"])]
        w = None if sorted_ else d_rgb.double().view(-1, 3)
        img, T = _exact_image(S, c64[0], case, clip, w, grads)
        shape = (case["height"], case["width"])
        out = dict(image=img.view(*shape, 3), T=T.view(shape), means=None, scales=None, quats=None,
                   opacities=None, sh=None)
        if sorted_:  # (the gradient in blend order has no dense form)
            return out
        leaves = {k: S[k].requires_grad_(True) for k in ("means", "scales", "quats", "sh")}
        with torch.no_grad():
            t0 = c64[0].project(S["means"])[3]
        rgb = _exact_rgb(leaves["means"], leaves["sh"], c64[0].centre(t0), case["sh"])
        M = _rotation(leaves["quats"]).transpose(1, 2) / leaves["scales"][:, :, None]
        g = torch.autograd.grad([rgb, M], list(leaves.values()), [grads[3], grads[1]])
        return dict(out, means=g[0] + grads[0], scales=g[1], quats=g[2], sh=g[3], opacities=grads[2])
    parts = [_exact_image(S, cam, case, None if clip is None else clip[i * px:(i + 1) * px]) for i, cam in enumerate(c64)]
    if case["entry"] == "serve":
        imgs, k = [p[0].view(case["height"], case["width"], 3) for p in parts], case["cams"]
        return dict(images=[imgs[i:i + k] for i in range(0, len(imgs), k)])
    return dict(rgb=torch.cat([p[0] for p in parts]), T=torch.cat([p[1] for p in parts]), n_contrib=None)
