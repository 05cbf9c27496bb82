"""Performance cases of the framework: what its users have it do, through
the public entry points of paper_2503_10855_amd.hx, over the sizes, options
and forms they use it with.

Kinds of case (the "kind" key):

image   one device image through Pipeline.edge_detect (mask and M), with
        the schedule the pipeline chooses by itself.
batch   a batch of device images through the batched call (masks and the
        images' M), descriptors marshalled once (prepare_batch), as a
        program that reuses its buffers does.
stages  the stage hook (B, L, Z, G, M and the mask) of one image.
srad    SRAD iterations on one image: the input is kept, a working copy
        is filtered in place.
serve   host images through a Server: every request submitted, then every
        mask collected.

Inputs: bright rectangles on noise (synth.image's recipe, drawn on the
GPU), for SRAD the same scene under multiplicative speckle noise.
"""
import math
import random

import numpy as np
import torch
import torch.nn.functional as F

from paper_2503_10855_amd import hx

# Blur sizes with the sigma each is used with.
SIGMA = {3: 0.8, 5: 1.0, 7: 1.5, 9: 2.0, 11: 2.5}
THETA = 0.1
LAMBDA = 0.5

# Bounds of the drawn cases: pixels of one image, pixels of one batch,
# pixels x iterations of one SRAD call.
MAX_IMAGE = 8192 * 8192
MAX_BATCH = 64 * 1920 * 1080
MAX_SRAD = 8192 * 8192 * 50


def listed():
    return [
        # One small frame: latency and launches are all of it.
        dict(name="image-256-k5", kind="image", h=256, w=256, k=5, pad=0),
        # One video frame at a time.
        dict(name="image-1080p-k5", kind="image", h=1080, w=1920, k=5, pad=0),
        # A crop of a larger image: odd sides, rows at the parent's pitch.
        dict(name="image-crop-701x1283-k3", kind="image", h=701, w=1283, k=3, pad=46),
        # One large image (a scan, a map tile) with the widest fused blur.
        dict(name="image-8192-k7", kind="image", h=8192, w=8192, k=7, pad=0),
        # A strongly smoothed frame: a blur wider than the fused sweeps take.
        dict(name="image-1080p-k9", kind="image", h=1080, w=1920, k=9, pad=0),
        # A clip of frames in one call: the throughput workload.
        dict(name="batch-64x1080p-k5", kind="batch", n=64, lo_h=1080, hi_h=1080,
             lo_w=1920, hi_w=1920, k=5),
        # A data set of photographs of every size in one call.
        dict(name="batch-256-uneven-k5", kind="batch", n=256, lo_h=64, hi_h=2048,
             lo_w=64, hi_w=2048, k=5),
        # Thumbnails: a small batch, where the launches weigh most.
        dict(name="batch-16-thumbs-k3", kind="batch", n=16, lo_h=64, hi_h=256,
             lo_w=64, hi_w=256, k=3),
        # The intermediate planes of a frame, for a program that uses them.
        dict(name="stages-1080p-k5", kind="stages", h=1080, w=1920, k=5, pad=0),
        # Despeckling one ultrasound-sized image: a chain of short kernels.
        dict(name="srad-512-100it", kind="srad", h=512, w=512, it=100, pad=0),
        # Despeckling one large radar image, resident in HBM.
        dict(name="srad-8192-50it", kind="srad", h=8192, w=8192, it=50, pad=0),
        # A burst of requests of mixed sizes at the server.
        dict(name="serve-48-mixed", kind="serve", n=48, lo=64, hi=1024, k=5),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _sides(rng, lo, hi, limit):
    """Two sides, each log-uniform in [lo, hi], of at most `limit` pixels."""
    while True:
        h, w = _log_int(rng, lo, hi), _log_int(rng, lo, hi)
        if h * w <= limit:
            return h, w


def draw(rng):
    kind = rng.choice(("image", "image", "image", "batch", "batch", "stages", "srad", "serve"))
    pad = rng.choice((0, 0, 0, 1, 4, 64, 333))
    if kind == "image":
        k = rng.choice((3, 5, 5, 5, 7, 7, 9, 11))
        h, w = _sides(rng, 64, 8192, MAX_IMAGE if k <= 7 else 1 << 23)
        return dict(kind=kind, h=h, w=w, k=k, pad=pad)
    if kind == "batch":
        # One size for every image (a clip) or a range of sizes (a set).
        k = rng.choice((3, 5, 5, 7))
        n = _log_int(rng, 2, 256)
        side = max(64, min(4096, int(math.sqrt(MAX_BATCH / n))))
        if rng.random() < 0.5:
            h, w = _sides(rng, 64, 2048, MAX_BATCH // n)
            return dict(kind=kind, n=n, lo_h=h, hi_h=h, lo_w=w, hi_w=w, k=k)
        lo, hi = 64, _log_int(rng, 128, max(129, side))
        return dict(kind=kind, n=n, lo_h=lo, hi_h=hi, lo_w=lo, hi_w=hi, k=k)
    if kind == "stages":
        h, w = _sides(rng, 64, 4096, 1 << 23)
        return dict(kind=kind, h=h, w=w, k=rng.choice((3, 5, 5, 7)), pad=pad)
    if kind == "srad":
        it = _log_int(rng, 5, 100)
        h, w = _sides(rng, 64, 8192, min(MAX_IMAGE, MAX_SRAD // it))
        return dict(kind=kind, h=h, w=w, it=it, pad=pad)
    return dict(kind=kind, n=_log_int(rng, 4, 64), lo=64, hi=_log_int(rng, 128, 1024), k=5)


# ---------------------------------------------------------------- inputs --
def _scene(h, w, seed, n_rect=8):
    """An h x w float32 device tensor: noise in [0, 0.2) and bright
    rectangles (sides a 16th to a quarter of the image's)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    img = torch.rand((h, w), generator=g, device="cuda") * 0.2
    r = random.Random(seed)
    for _ in range(n_rect):
        rw, rh = r.randint(max(1, w // 16), max(1, w // 4)), r.randint(max(1, h // 16),
                                                                       max(1, h // 4))
        x0, y0 = r.randint(0, w - rw), r.randint(0, h - rh)
        img[y0:y0 + rh, x0:x0 + rw] = r.uniform(0.5, 1.0)
    return img


def _speckled(h, w, seed):
    """The scene times gamma(4, 1/4) noise (mean 1), plus 0.05."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + 1)
    s = torch.zeros((h, w), device="cuda")
    for _ in range(4):
        s -= torch.rand((h, w), generator=g, device="cuda").clamp_(min=1e-6).log_()
    return _scene(h, w, seed) * (0.25 * s) + 0.05


def _pitched(img, pad):
    """The image as columns of a wider buffer (a crop) when pad > 0."""
    if not pad:
        return img
    buf = torch.zeros((img.shape[0], img.shape[1] + pad), dtype=img.dtype, device=img.device)
    view = buf[:, :img.shape[1]]
    view.copy_(img)
    return view


def _n_rect(h, w):
    return 64 if h * w >= 1 << 24 else 8


def _batch_sizes(case):
    """The batch's image sizes: a property of the case, not of the seed."""
    r = random.Random(case["n"] * 1000003 + case["hi_h"] * 4099 + case["hi_w"])
    out, left = [], MAX_BATCH
    for _ in range(case["n"]):
        h, w = (_log_int(r, case["lo_h"], case["hi_h"]), _log_int(r, case["lo_w"], case["hi_w"]))
        if h * w > left:
            break
        out.append((h, w))
        left -= h * w
    return out


def _batch_images(case, seed):
    """The images as views of one buffer, each on a 256-byte boundary."""
    sizes = _batch_sizes(case)
    at = [0]
    for h, w in sizes:
        at.append(at[-1] + (h * w + 63) // 64 * 64)
    buf = torch.zeros(at[-1], device="cuda")
    imgs = [buf[o:o + h * w].view(h, w) for o, (h, w) in zip(at, sizes)]
    for i, (im, (h, w)) in enumerate(zip(imgs, sizes)):
        im.copy_(_scene(h, w, seed * 1009 + i))
    return buf, imgs, at


def _serve_sizes(case):
    r = random.Random(case["n"] * 7919 + case["hi"])
    return [(_log_int(r, case["lo"], case["hi"]), _log_int(r, case["lo"], case["hi"]))
            for _ in range(case["n"])]


class _Served:
    """A server with its pipeline, closed with the program's last use of it."""

    def __init__(self, k):
        self.p = hx.Pipeline(ksize=k, sigma=SIGMA[k], theta=THETA, max_pixels=1 << 25,
                             max_images=64, forms=hx.FORM_BATCH, batch_contexts=4)
        self.srv = hx.Server(self.p, hbm_budget=self.p.memory()[0] + (512 << 20), streams=4,
                             max_batch=64)

    def __del__(self):
        self.srv.close()
        self.p.close()


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("image", "stages"):
        h, w, k = case["h"], case["w"], case["k"]
        src = _pitched(_scene(h, w, seed, _n_rect(h, w)), case["pad"])
        p = hx.Pipeline(ksize=k, sigma=SIGMA[k], theta=THETA, max_pixels=h * w, max_images=1)
        mask = _pitched(torch.zeros((h, w), dtype=torch.uint8, device="cuda"), case["pad"])
        return dict(kind=kind, p=p, src=src, mask=mask, M=torch.zeros(1, device="cuda"))
    if kind == "batch":
        k = case["k"]
        buf, imgs, at = _batch_images(case, seed)
        n = len(imgs)
        p = hx.Pipeline(ksize=k, sigma=SIGMA[k], theta=THETA, max_pixels=sum(i.numel() for i in imgs),
                        max_images=n, forms=hx.FORM_BATCH)
        masks = torch.zeros(at[-1], dtype=torch.uint8, device="cuda")
        views = [masks[o:o + i.numel()].view(i.shape) for o, i in zip(at, imgs)]
        M = torch.zeros(n, device="cuda")
        return dict(kind=kind, p=p, plan=p.prepare_batch(imgs, views, M), masks=masks, M=M)
    if kind == "srad":
        h, w = case["h"], case["w"]
        src = _pitched(_speckled(h, w, seed), case["pad"])
        p = hx.Pipeline(max_pixels=h * w, max_images=1, forms=hx.FORM_SRAD)
        return dict(kind=kind, p=p, src=src, J=_pitched(torch.empty_like(src), case["pad"]),
                    it=case["it"], q=torch.zeros(case["it"], dtype=torch.float64, device="cuda"))
    pool = _scene(2048, 2048, seed, 16).cpu().numpy()
    r = random.Random(seed)
    crops = []
    for h, w in _serve_sizes(case):
        y0, x0 = r.randint(0, 2048 - h), r.randint(0, 2048 - w)
        crops.append(pool[y0:y0 + h, x0:x0 + w])
    return dict(kind=kind, served=_Served(case["k"]), crops=crops,
                out=[np.zeros(c.shape, np.uint8) for c in crops])


# ------------------------------------------------------------------- run --
def run(s):
    kind = s["kind"]
    if kind == "image":
        return {"mask": s["p"].edge_detect(s["src"], mask=s["mask"], dmax=s["M"]), "M": s["M"]}
    if kind == "batch":
        s["plan"].run()
        return {"masks": s["masks"], "M": s["M"]}
    if kind == "stages":
        return s["p"].edge_detect_stages(s["src"])
    if kind == "srad":
        s["J"].copy_(s["src"])
        return {"J": s["p"].srad(s["J"], s["it"], LAMBDA, q_log=s["q"]), "q": s["q"]}
    srv = s["served"].srv
    tickets = [srv.submit(c) for c in s["crops"]]
    for t, c, m in zip(tickets, s["crops"], s["out"]):
        while srv.poll(t, c.shape, out=m) is None:
            pass
    return s["out"]


# ------------------------------------------------------------------ work --
def work(case):
    """Each input read once, each output written once; the additions and
    multiplications of the separable blur, Sobel, Laplacian and threshold
    (2k + 11 and, per SRAD iteration, 38 per pixel)."""
    kind = case["kind"]
    if kind in ("image", "stages"):
        px = case["h"] * case["w"]
        return {"bytes": px * (5 if kind == "image" else 18), "flops": px * (2 * case["k"] + 11)}
    if kind == "batch":
        px = sum(h * w for h, w in _batch_sizes(case))
        return {"bytes": 5 * px, "flops": px * (2 * case["k"] + 11)}
    if kind == "srad":
        # Every iteration depends on a sum over the whole image before it:
        # the image is read and written once per iteration.
        px = case["h"] * case["w"]
        return {"bytes": 8 * px * (case["it"] + 1), "flops": 38 * px * case["it"]}
    px = sum(h * w for h, w in _serve_sizes(case))
    return {"bytes": 5 * px, "flops": px * (2 * case["k"] + 11)}


# ----------------------------------------------------------------- exact --
def _edge64(img, k):
    """B, L, G and M of one image in float64 (every stage reads its input at
    clamped coordinates)."""
    x = img.double()[None, None]
    r = k // 2
    g = torch.arange(-r, r + 1, dtype=torch.float64, device=x.device)
    g = torch.exp(-g * g / (2.0 * SIGMA[k] ** 2))
    g = g / g.sum()
    p = F.pad(x, (r, r, r, r), mode="replicate")
    h, w = img.shape
    p = sum(g[i] * p[..., i:i + w] for i in range(k))
    b = sum(g[i] * p[:, :, i:i + h] for i in range(k))
    q = F.pad(b, (1, 1, 1, 1), mode="replicate")[0, 0]
    at = lambda dy, dx: q[1 + dy:1 + dy + h, 1 + dx:1 + dx + w]  # noqa: E731
    lap = at(-1, 0) + at(1, 0) + at(0, -1) + at(0, 1) - 4.0 * at(0, 0)
    gx = (at(-1, 1) + 2 * at(0, 1) + at(1, 1)) - (at(-1, -1) + 2 * at(0, -1) + at(1, -1))
    gy = (at(1, -1) + 2 * at(1, 0) + at(1, 1)) - (at(-1, -1) + 2 * at(-1, 0) + at(-1, 1))
    mag = torch.sqrt(gx * gx + gy * gy)
    return b[0, 0], lap, mag, mag.max().reshape(1)


def _srad64(img, niter):
    j = img.double()
    q = torch.zeros(niter, dtype=torch.float64, device=j.device)
    for it in range(niter):
        m = j.mean()
        q0 = (j * j).mean() / (m * m) - 1.0
        q[it] = q0
        n = torch.cat((j[:1], j[:-1])) - j
        s = torch.cat((j[1:], j[-1:])) - j
        w = torch.cat((j[:, :1], j[:, :-1]), 1) - j
        e = torch.cat((j[:, 1:], j[:, -1:]), 1) - j
        g2 = (n * n + s * s + w * w + e * e) / (j * j)
        lap = (n + s + w + e) / j
        qs = (0.5 * g2 - lap * lap / 16.0) / (1.0 + 0.25 * lap) ** 2
        c = (1.0 / (1.0 + (qs - q0) / (q0 * (1.0 + q0)))).clamp(0.0, 1.0)
        c = torch.where(q0 > 0, c, torch.ones_like(c))
        del g2, lap, qs
        d = c * (n + w)
        d += torch.cat((c[1:], c[-1:])) * s
        d += torch.cat((c[:, 1:], c[:, -1:]), 1) * e
        j = j + 0.25 * LAMBDA * d
    return j, q


def exact(case, seed):
    """Masks and Z are decisions, not computed numbers: None."""
    kind = case["kind"]
    if kind in ("image", "stages"):
        h, w, k = case["h"], case["w"], case["k"]
        b, lap, mag, m = _edge64(_scene(h, w, seed, _n_rect(h, w)), k)
        if kind == "image":
            return {"mask": None, "M": m}
        return {"M": m, "mask": None, "B": b, "L": lap, "Z": None, "G": mag}
    if kind == "batch":
        _, imgs, _ = _batch_images(case, seed)
        return {"masks": None, "M": torch.cat([_edge64(i, case["k"])[3] for i in imgs])}
    if kind == "srad":
        j, q = _srad64(_speckled(case["h"], case["w"], seed), case["it"])
        return {"J": j, "q": q}
    return None
