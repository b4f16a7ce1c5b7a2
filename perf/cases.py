"""Performance cases: what a user of the package has it do, over the real range.

Every case goes through the package's public entry points (``segment``,
``Context``, ``Batch``, ``warm.warm_segment``, ``warm.Net.train_step``), on
synthetic images of the benchmark's kind: a Voronoi partition, each region
painted with a colour and a linear ramp, plus Gaussian noise.

Kinds
  frame    one image, one call (``segment``): the image is new on every call
           of a real program, the workspace is kept
  video    a frame started from the previous frame's centres, two rounds
  context  the step-by-step interface: rounds until the centres rest, then
           the stray-pixel filter, then the results
  batch    many images through one plan (one graph)
  warm     a frame started from the trained net's labels
  train    one training step of that net
"""
import math

import torch

import paper_1509_04232_amd as slic

DEV = "cuda"


def listed():
    return [
        # the smallest call: a thumbnail or a region of interest, every output;
        # time is launches and latency
        dict(name="thumb_96x72", kind="frame", w=96, h=72, S=8, K=0, m=10.0, iters=3, perturb=True,
             enforce=True, centres=True, energy=True, channels=3, pad=0, color="lab",
             squared=False, sigma=8.0),
        # a preview of a camera stream, labels only, few rounds, no clean-up
        dict(name="preview_320x240", kind="frame", w=320, h=240, S=16, K=0, m=10.0, iters=5,
             perturb=False, enforce=False, centres=False, energy=False, channels=3, pad=0,
             color="lab", squared=False, sigma=8.0),
        # the headline: one camera frame with clean-up
        dict(name="camera_640x480", kind="frame", w=640, h=480, S=16, K=0, m=10.0, iters=10,
             perturb=True, enforce=True, centres=False, energy=False, channels=3, pad=0,
             color="lab", squared=False, sigma=8.0),
        # a full-HD frame with a dense grid and strong noise
        dict(name="hd_1920x1080", kind="frame", w=1920, h=1080, S=8, K=0, m=10.0, iters=10,
             perturb=True, enforce=True, centres=False, energy=False, channels=3, pad=0,
             color="lab", squared=False, sigma=12.0),
        # a photograph by its number of superpixels: odd width, odd step (27)
        dict(name="photo_933x800_k1000", kind="frame", w=933, h=800, S=0, K=1000, m=10.0, iters=10,
             perturb=True, enforce=True, centres=True, energy=False, channels=3, pad=0,
             color="lab", squared=False, sigma=8.0),
        # the largest photograph: 14 megapixels, odd in both directions, step 84
        dict(name="photo_3631x3859_k2000", kind="frame", w=3631, h=3859, S=0, K=2000, m=10.0,
             iters=10, perturb=True, enforce=True, centres=False, energy=False, channels=3, pad=0,
             color="lab", squared=False, sigma=8.0),
        # step by step on four-byte pixels with padded rows: rounds until the
        # centres rest, the stray-pixel filter, labels and centres
        dict(name="context_1024x1024_rgbx", kind="context", w=1024, h=1024, S=0, K=1000, m=20.0,
             iters=10, threshold=1.5, passes=2, perturb=True, channels=4, pad=64, color="lab",
             squared=False, sigma=8.0),
        # a live stream: this frame from the last one's centres
        dict(name="video_640x480", kind="video", w=640, h=480, S=16, K=0, m=10.0, iters=2,
             channels=3, pad=0, sigma=8.0),
        # throughput: 64 images of mixed sizes and steps through one plan
        dict(name="batch_mixed_64", kind="batch", count=64, mixed=True, w=1920, h=1080, S=16,
             m=10.0, iters=10, enforce=False, pick=4),
        # throughput: 16 camera frames with clean-up
        dict(name="batch_camera_16", kind="batch", count=16, mixed=False, w=640, h=480, S=16,
             m=10.0, iters=10, enforce=True, pick=0),
        # a full-HD frame from the trained net's labels, four rounds
        dict(name="warm_1920x1080", kind="warm", w=1920, h=1080, S=16, m=10.0, iters=4,
             confidence=0.8, enforce=False, energy=True, sigma=8.0),
        # training the net: forward and backward on a batch of crops, and Adam
        dict(name="train_32x128x128", kind="train", crops=32, cw=128, ch=128, S=16),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """Width and height: the pixel count spread over its logarithm, odd sides
    as often as even ones, half the widths multiples of four."""
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    aspect = rng.choice([4 / 3, 16 / 9, 1.0, 3 / 4]) * rng.uniform(0.9, 1.1)
    w = max(48, int(math.sqrt(n * aspect)))
    if rng.random() < 0.5:
        w = (w + 3) // 4 * 4
    return w, max(48, int(n / w))


def draw(rng):
    kind = rng.choice(["frame"] * 6 + ["video", "context", "batch", "warm", "warm", "train"])
    if kind == "frame":
        w, h = _size(rng, 96 * 72, 2200 * 1300)
        by_count = rng.random() < 0.4
        return dict(kind="frame", w=w, h=h, S=0 if by_count else rng.choice([8, 16, 32]),
                    K=_log_int(rng, max(8, w * h // 4096), w * h // 100) if by_count else 0,
                    m=rng.choice([5.0, 10.0, 20.0]), iters=rng.randint(3, 10),
                    perturb=rng.random() < 0.8, enforce=rng.random() < 0.7,
                    centres=rng.random() < 0.5, energy=rng.random() < 0.3,
                    channels=rng.choice([3, 3, 4]), pad=rng.choice([0, 0, 0, 13, 64]),
                    color=rng.choice(["lab"] * 6 + ["rgb", "xyz"]),
                    squared=rng.random() < 0.15, sigma=rng.choice([4.0, 8.0, 12.0]))
    if kind == "video":
        w, h = _size(rng, 160 * 120, 1920 * 1080)
        return dict(kind="video", w=w, h=h, S=rng.choice([8, 16, 32]), K=0, m=10.0,
                    iters=rng.randint(1, 3), channels=rng.choice([3, 4]), pad=0, sigma=8.0)
    if kind == "context":
        w, h = _size(rng, 160 * 120, 1920 * 1080)
        return dict(kind="context", w=w, h=h, S=0, K=_log_int(rng, max(16, w * h // 4096), w * h // 100),
                    m=rng.choice([10.0, 20.0]), iters=rng.randint(4, 12),
                    threshold=rng.choice([0.5, 1.5, 3.0]), passes=rng.randint(1, 3), perturb=True,
                    channels=rng.choice([3, 4]), pad=rng.choice([0, 64]), color="lab",
                    squared=rng.random() < 0.2, sigma=8.0)
    if kind == "batch":
        mixed = rng.random() < 0.5
        w, h = _size(rng, 160 * 120, 800 * 600)
        return dict(kind="batch", count=rng.randint(2, 24), mixed=mixed, w=w, h=h,
                    S=rng.choice([8, 16, 32]), m=10.0, iters=rng.randint(4, 10),
                    enforce=rng.random() < 0.5, pick=rng.randint(0, 1 << 20))
    if kind == "warm":
        w, h = _size(rng, 160 * 120, 1920 * 1080)
        return dict(kind="warm", w=w, h=h, S=rng.choice([8, 16, 24, 32]), m=10.0,
                    iters=rng.randint(2, 4), confidence=rng.choice([0.7, 0.75, 0.8]),
                    enforce=rng.random() < 0.5, energy=True, sigma=8.0)
    return dict(kind="train", crops=_log_int(rng, 2, 32), cw=rng.randint(48, 144),
                ch=rng.randint(48, 128), S=rng.choice([8, 16, 24]))


# ----------------------------------------------------------------- inputs

def _gen(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + salt * 7919 + 17) % (1 << 62))
    return g


def _image(w, h, sigma, g, regions=None):
    """uint8 (h, w, 3): regions of one colour and a ramp each, plus noise."""
    regions = regions or max(2, min(4096, w * h // 1200))
    sx = torch.rand(regions, generator=g, device=DEV) * w
    sy = torch.rand(regions, generator=g, device=DEV) * h
    col = torch.rand((regions, 3), generator=g, device=DEV) * 255.0
    ang = torch.rand(regions, generator=g, device=DEV) * (2.0 * math.pi)
    reach = math.sqrt(w * h / (math.pi * regions))
    xs = torch.arange(w, device=DEV, dtype=torch.float32)
    out = torch.empty((h, w, 3), dtype=torch.uint8, device=DEV)
    step = max(1, (1 << 27) // (w * regions))
    dx2 = (xs[:, None] - sx[None, :]) ** 2  # (w, regions)
    for y0 in range(0, h, step):
        ys = torch.arange(y0, min(h, y0 + step), device=DEV, dtype=torch.float32)
        dy2 = (ys[:, None] - sy[None, :]) ** 2
        r = (dx2[None, :, :] + dy2[:, None, :]).argmin(2)  # (rows, w)
        along = (xs[None, :] - sx[r]) * torch.cos(ang[r]) + (ys[:, None] - sy[r]) * torch.sin(ang[r])
        ramp = 20.0 * (along / reach).clamp(-1.0, 1.0)
        noise = torch.randn((len(ys), w, 3), generator=g, device=DEV) * sigma
        out[y0:y0 + len(ys)] = (col[r] + ramp[..., None] + noise).round().clamp(0, 255).to(torch.uint8)
    return out


def _pack(img, channels, pad):
    """The flat pixel buffer of an image: 3 or 4 bytes a pixel, padded rows."""
    h, w, _ = img.shape
    if channels == 3 and not pad:
        return img.reshape(-1).contiguous(), None
    pitch = w * channels + pad
    buf = torch.zeros((h, pitch), dtype=torch.uint8, device=DEV)
    buf[:, :w * channels].view(h, w, channels)[:, :, :3] = img
    return buf.reshape(-1), pitch


def _params(c, pitch=None):
    return slic.Params(c["w"], c["h"], S=c.get("S", 0), K=c.get("K", 0), m=c["m"],
                       perturb=c.get("perturb", True), channels=c.get("channels", 3), pitch=pitch,
                       color=c.get("color", "lab"), squared_distance=c.get("squared", False))


def _step(c):
    if c.get("S", 0) > 0:
        return c["S"]
    return max(1, int(math.floor(math.sqrt(c["w"] * c["h"] / c["K"]) + 0.5)))


def _cells(w, h, S):
    return -(-w // S), -(-h // S)


_SIZES = [(320, 240), (640, 480), (1280, 720), (1920, 1080)]


def _batch_shapes(c):
    """(w, h, S) of every image: camera-like sizes and steps, or one shape."""
    if not c["mixed"]:
        return [(c["w"], c["h"], c["S"])] * c["count"]
    g = torch.Generator().manual_seed(c["pick"])
    at = torch.randint(0, 12, (c["count"],), generator=g).tolist()
    return [_SIZES[a % 4] + ((8, 16, 32)[a // 4],) for a in at]


def _net_params(S, g):
    """A net as training leaves it: He-scaled convolutions, a phase bias that
    favours the cell whose middle is nearest."""
    o = slic.warm.offsets(S)
    p = torch.zeros(o["end"], device=DEV)
    for name, nxt, fan, scale in (("W1", "b1", 3, 1.0), ("W2", "b2", 32, 1.0), ("W3", "b3", 32, 0.15)):
        n = o[nxt] - o[name]
        p[o[name]:o[nxt]] = torch.randn(n, generator=g, device=DEV) * (scale * math.sqrt(2.0 / (9 * fan)))
    for name, nxt in (("b1", "W2"), ("b2", "W3"), ("b3", "P")):
        p[o[name]:o[nxt]] = torch.randn(o[nxt] - o[name], generator=g, device=DEV) * 0.05
    at = (torch.arange(S, device=DEV) + 0.5) / S - 0.5
    off = torch.tensor([-1.0, 0.0, 1.0], device=DEV)
    d2 = ((at[:, None, None, None] - off[None, None, :, None]) ** 2 +
          (at[None, :, None, None] - off[None, None, None, :]) ** 2)  # (y, x, dy, dx)
    p[o["P"]:] = (-7.0 * d2).reshape(-1)
    return p


def _train_images(c, seed):
    """Four images' CIELAB planes (float32) and label maps near convergence:
    each pixel's nearest of the nine jittered cell centres."""
    out = []
    S = c["S"]
    for i in range(4):
        g = _gen(seed, 100 + i)
        w, h = max(640, c["cw"]), max(480, c["ch"])
        img = _image(w, h, 8.0, g, 256)
        lab = [t.float().contiguous() for t in _planes64(img, "lab")]
        ncx, ncy = _cells(w, h, S)
        cen = torch.zeros((ncx * ncy, 5), dtype=torch.float64, device=DEV)
        k = torch.arange(ncx * ncy, device=DEV)
        jit = torch.rand((2, ncx * ncy), generator=g, device=DEV).double() - 0.5
        cen[:, 3] = (k % ncx + 0.5 + 0.6 * jit[0]) * S
        cen[:, 4] = (k // ncx + 0.5 + 0.6 * jit[1]) * S
        flat = [torch.zeros((h, w), dtype=torch.float64, device=DEV)] * 3
        labels = _associate64(flat, S, 1.0, cen, False)[0].to(torch.int32)
        out.append((*lab, labels))
    return out


def _train_origins(c, images, seed):
    g = torch.Generator().manual_seed(int(seed) * 31 + 5)
    got = []
    for _ in range(c["crops"]):
        i, u, v = (float(t) for t in torch.rand(3, generator=g))
        h, w = images[0][0].shape
        got.append((int(i * len(images)), int(u * (w - c["cw"] + 1)), int(v * (h - c["ch"] + 1))))
    return got


def _moments(n, g):
    """Adam's moments some steps into training."""
    return (torch.randn(n, generator=g, device=DEV) * 1e-3,
            (torch.rand(n, generator=g, device=DEV) + 0.5) * 1e-6)


_TRAIN_STEP, _TRAIN_LR = 200, 2e-3


def _video_frames(c, seed):
    """Two views of one canvas, shifted by up to two pixels."""
    img = _image(c["w"] + 4, c["h"] + 4, c["sigma"], _gen(seed))
    s = int(seed) % 25
    a = img[2:2 + c["h"], 2:2 + c["w"]].contiguous()
    b = img[s % 5:s % 5 + c["h"], s // 5:s // 5 + c["w"]].contiguous()
    return a, b


def _video_centres(c, before):
    planes = _planes64(before, "lab")
    S = _step(c)
    cen = _seeds64(planes, S, True)
    for _ in range(10):
        labels, _ = _associate64(planes, S, c["m"] / S, cen, False)
        cen = _means64(planes, labels, cen)
    return cen.float().contiguous()


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind in ("frame", "context"):
        rgb, pitch = _pack(_image(c["w"], c["h"], c["sigma"], _gen(seed)), c["channels"], c["pad"])
        p = _params(c, pitch)
        return dict(case=c, rgb=rgb, p=p, ws=slic.workspace_for(p))
    if kind == "video":
        before, now = _video_frames(c, seed)
        rgb, pitch = _pack(now, c["channels"], c["pad"])
        p = _params(c, pitch)
        return dict(case=c, rgb=rgb, p=p, ws=slic.workspace_for(p), cen=_video_centres(c, before))
    if kind == "batch":
        shapes = _batch_shapes(c)
        params = [slic.Params(w, h, S=S, m=c["m"]) for w, h, S in shapes]
        images = [_image(w, h, 8.0, _gen(seed, i)).reshape(-1) for i, (w, h, S) in enumerate(shapes)]
        return dict(case=c, batch=slic.Batch(params, images, c["iters"], c["enforce"]))
    if kind == "warm":
        rgb, _ = _pack(_image(c["w"], c["h"], c["sigma"], _gen(seed)), 3, 0)
        p = _params(c)
        net = slic.warm.prepare(_net_params(c["S"], _gen(seed, 1)), c["S"], c["confidence"])
        return dict(case=c, rgb=rgb, p=p, net=net, ws=slic.workspace_for(p))
    images = _train_images(c, seed)
    g = _gen(seed, 2)
    net = slic.warm.Net(c["S"], c["crops"], c["cw"], c["ch"],
                        params=_net_params(c["S"], g).cpu().numpy())
    m, v = _moments(net.count, g)
    net.m.copy_(m)
    net.v.copy_(v)
    net.steps = _TRAIN_STEP
    crops = [slic.warm.crop(*images[i][:3], x, y, images[i][3])
             for i, x, y in _train_origins(c, images, seed)]
    return dict(case=c, net=net, crops=crops, images=images)


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "frame":
        return slic.segment(state["rgb"], state["p"], c["iters"], enforce=c["enforce"],
                            want_centres=c["centres"], want_energy=c["energy"],
                            workspace=state["ws"])
    if kind == "video":
        ctx = slic.Context(state["p"], state["rgb"], centres=state["cen"], workspace=state["ws"])
        ctx.iterate(c["iters"])
        labels = ctx.labels()
        centres, counts = ctx.centres()
        ctx.close()
        return dict(labels=labels, centres=centres, counts=counts)
    if kind == "context":
        ctx = slic.Context(state["p"], state["rgb"], workspace=state["ws"])
        rounds = ctx.iterate_converge(c["iters"], c["threshold"])
        energy = ctx.energy()
        ctx.filter_stray(c["passes"])
        labels = ctx.labels()
        centres, counts = ctx.centres()
        ctx.close()
        return dict(rounds=rounds, energy=energy, labels=labels, centres=centres, counts=counts)
    if kind == "batch":
        b = state["batch"].run()
        return dict(labels=b.labels, n_segments=b.n_segments)
    if kind == "warm":
        return slic.warm.warm_segment(state["rgb"], state["p"], state["net"], c["iters"],
                                      enforce=c["enforce"], want_energy=c["energy"],
                                      workspace=state["ws"])
    net = state["net"]
    loss = net.train_step(state["crops"], _TRAIN_LR)
    return dict(loss=loss, grad=net.grad, params=net.params, m=net.m, v=net.v)


# ------------------------------------------------------------------- work

_CONV_FLOPS = 2 * 9 * (3 * 32 + 32 * 32 + 32 * 9)  # the net's three layers, per pixel
_ASSOC_OPS = 166                                   # Eq. 1 for nine centres and the sums


def work(case):
    """Each input once in, each output once out; the arithmetic of Eq. 1 and
    of the convolutions."""
    c, kind = case, case["kind"]
    if kind == "train":
        n = c["crops"] * c["cw"] * c["ch"]
        count = 9 * (3 * 32 + 32 * 32 + 32 * 9) + 73 + 9 * c["S"] ** 2
        return dict(bytes=n * (12 + 4) + count * 4 * 8, flops=n * 3 * _CONV_FLOPS)
    shapes = _batch_shapes(c) if kind == "batch" else [(c["w"], c["h"], _step(c))]
    rounds = 1 + (c["iters"] if kind != "context" else 1)
    b = f = 0
    for w, h, S in shapes:
        n = w * h
        ncx, ncy = _cells(w, h, S)
        b += n * (c.get("channels", 3) + 4)
        f += n * _ASSOC_OPS * rounds
        if c.get("centres") or kind in ("video", "context"):
            b += ncx * ncy * 24
        if kind == "video":
            b += ncx * ncy * 20
        if kind == "warm":
            f += n * _CONV_FLOPS
    return dict(bytes=b, flops=f)


# ------------------------------------------------- the same in 64 bits

def _planes64(img, color):
    """CIELAB (or XYZ x 100, or the bytes) planes of an image, float64."""
    v = img[..., :3].double()
    if color == "rgb":
        return [v[..., i] for i in range(3)]
    v = v / 255.0
    lin = torch.where(v <= 0.04045, v / 12.92, ((v + 0.055) / 1.055) ** 2.4)
    m = torch.tensor([[0.4124, 0.3576, 0.1805], [0.2126, 0.7152, 0.0722],
                      [0.0193, 0.1192, 0.9505]], dtype=torch.float64, device=img.device)
    m = m / m.sum(1, keepdim=True)
    xyz = [sum(m[i, j] * lin[..., j] for j in range(3)) for i in range(3)]
    if color == "xyz":
        return [100.0 * t for t in xyz]
    fx, fy, fz = (torch.where(t > 216 / 24389, t.clamp_min(1e-12) ** (1 / 3),
                              (24389 / 27 * t + 16.0) / 116.0) for t in xyz)
    return [116.0 * fy - 16.0, 500.0 * (fx - fy), 200.0 * (fy - fz)]


def _seeds64(planes, S, perturb):
    h, w = planes[0].shape
    ncx, ncy = _cells(w, h, S)

    def middles(n, extent):
        lo = torch.arange(n, device=DEV) * S
        return lo + ((lo + S).clamp_max(extent) - lo - 1) // 2
    x = middles(ncx, w).repeat(ncy)
    y = middles(ncy, h).repeat_interleave(ncx)
    if perturb:
        grad = torch.zeros_like(planes[0])
        xi, yi = torch.arange(w, device=DEV), torch.arange(h, device=DEV)
        for p in planes:
            gx = p[:, (xi + 1).clamp_max(w - 1)] - p[:, (xi - 1).clamp_min(0)]
            gy = p[(yi + 1).clamp_max(h - 1)] - p[(yi - 1).clamp_min(0)]
            grad += gx * gx + gy * gy
        bx, by, best = x, y, grad[y, x]
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                nx, ny = x + dx, y + dy
                ok = (nx >= 0) & (ny >= 0) & (nx < w) & (ny < h)
                v = grad[ny.clamp(0, h - 1), nx.clamp(0, w - 1)]
                ok &= v < best
                bx, by, best = torch.where(ok, nx, bx), torch.where(ok, ny, by), torch.where(ok, v, best)
        x, y = bx, by
    return torch.stack([p[y, x] for p in planes] + [x.double(), y.double()], 1)


def _associate64(planes, S, wgt, cen, squared):
    """(labels (h, w), their distance): the nearest of the nine centres."""
    h, w = planes[0].shape
    ncx, ncy = _cells(w, h, S)
    x = torch.arange(w, device=DEV)[None, :].expand(h, w)
    y = torch.arange(h, device=DEV)[:, None].expand(h, w)
    best = torch.full((h, w), math.inf, dtype=torch.float64, device=DEV)
    label = torch.zeros((h, w), dtype=torch.int64, device=DEV)
    for dy in (-1, 0, 1):
        for dx in (-1, 0, 1):
            cx, cy = x // S + dx, y // S + dy
            ok = (cx >= 0) & (cy >= 0) & (cx < ncx) & (cy < ncy)
            k = cy.clamp(0, ncy - 1) * ncx + cx.clamp(0, ncx - 1)
            q = cen[k]
            s = sum((q[..., i] - planes[i]) ** 2 for i in range(3))
            t = (q[..., 3] - x) ** 2 + (q[..., 4] - y) ** 2
            d = s + wgt * wgt * t if squared else s.sqrt() + wgt * t.sqrt()
            ok &= d < best
            best, label = torch.where(ok, d, best), torch.where(ok, k, label)
    return label, best


def _means64(planes, labels, cen, votes=None):
    """The mean of each centre's pixels (in whole steps of 2^-24, so that the
    order of the additions does not matter); one without pixels stays."""
    h, w = planes[0].shape
    at = labels.reshape(-1)
    x = torch.arange(w, device=DEV)[None, :].expand(h, w)
    y = torch.arange(h, device=DEV)[:, None].expand(h, w)
    rows = [(p * 2.0 ** 24).round().to(torch.int64) for p in planes] + [x << 24, y << 24]
    keep = torch.ones_like(at) if votes is None else votes.reshape(-1).to(torch.int64)
    n = torch.zeros(len(cen), dtype=torch.int64, device=DEV).index_add_(0, at, keep)
    out = cen.clone()
    for j, r in enumerate(rows):
        s = torch.zeros(len(cen), dtype=torch.int64, device=DEV).index_add_(0, at, r.reshape(-1) * keep)
        out[:, j] = torch.where(n > 0, s.double() / n.clamp_min(1) / 2.0 ** 24, cen[:, j])
    return out


def _net64(planes, params, S, ox=0, oy=0, valid=None):
    """The net's logits (h, w, 9) in float64, zero padding at the borders."""
    o = slic.warm.offsets(S)
    h, w = planes[0].shape
    inside = torch.ones((h, w, 1), dtype=torch.float64, device=DEV) if valid is None else valid[..., None]
    a = torch.stack([planes[0] / 100.0, planes[1] / 128.0, planes[2] / 128.0], -1) * inside
    for layer, (wn, bn, nxt, cin, cout) in enumerate((("W1", "b1", "W2", 3, 32), ("W2", "b2", "W3", 32, 32),
                                                      ("W3", "b3", "P", 32, 9))):
        wt = params[o[wn]:o[bn]].reshape(9, cout, cin)
        pad = torch.nn.functional.pad(a, (0, 0, 1, 1, 1, 1))
        z = params[o[bn]:o[nxt]].expand(h, w, cout)
        for t in range(9):
            z = z + pad[t // 3:t // 3 + h, t % 3:t % 3 + w] @ wt[t].T
        a = torch.relu(z) * inside if layer < 2 else z
    ph = ((torch.arange(h, device=DEV) + oy) % S)[:, None] * S + ((torch.arange(w, device=DEV) + ox) % S)[None, :]
    return a + params[o["P"]:].reshape(S * S, 9)[ph]


def _warm_labels64(planes, params, S, confidence):
    h, w = planes[0].shape
    ncx, ncy = _cells(w, h, S)
    prob = torch.softmax(_net64(planes, params, S), -1)
    p, cls = prob.max(-1)
    cx = (torch.arange(w, device=DEV)[None, :] // S + cls % 3 - 1).clamp(0, ncx - 1)
    cy = (torch.arange(h, device=DEV)[:, None] // S + cls // 3 - 1).clamp(0, ncy - 1)
    return cy * ncx + cx, p >= confidence


def _train64(c, seed):
    images = _train_images(c, seed)
    g = _gen(seed, 2)
    S = c["S"]
    p = _net_params(S, g)
    m, v = (t.double() for t in _moments(len(p), g))
    p = p.double().requires_grad_(True)
    grad = torch.zeros_like(p)
    total, count = 0.0, 0
    for i, ox, oy in _train_origins(c, images, seed):
        L, A, B, labels = images[i]
        h, w = L.shape
        ncx = _cells(w, h, S)[0]
        part = [t[oy:oy + c["ch"], ox:ox + c["cw"]] for t in (L, A, B, labels)]
        k = part[3].long()
        dy = k // ncx - (torch.arange(c["ch"], device=DEV) + oy)[:, None] // S
        dx = k % ncx - (torch.arange(c["cw"], device=DEV) + ox)[None, :] // S
        ok = (dx.abs() <= 1) & (dy.abs() <= 1)
        target = ((dy + 1) * 3 + dx + 1)[ok]
        z = _net64([t.double() for t in part[:3]], p, S, ox, oy)
        loss = torch.nn.functional.cross_entropy(z[ok], target, reduction="sum")
        grad += torch.autograd.grad(loss, p)[0]
        total, count = total + float(loss.detach()), count + len(target)
    grad = grad / count
    step = _TRAIN_STEP + 1
    m, v = 0.9 * m + 0.1 * grad, 0.999 * v + 0.001 * grad * grad
    new = p.detach() - _TRAIN_LR * (m / (1 - 0.9 ** step)) / ((v / (1 - 0.999 ** step)).sqrt() + 1e-8)
    loss = torch.tensor([total / count], dtype=torch.float64)
    return dict(loss=loss, grad=grad, params=new, m=m, v=v)


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "train":
        return _train64(c, seed)
    if kind == "batch" or not (kind in ("video", "context", "warm") or c["centres"] or c["energy"]):
        return None  # whole numbers only
    S, squared = _step(c), c.get("squared", False)
    wgt = c["m"] / S
    if kind == "video":
        before, img = _video_frames(c, seed)
        planes = _planes64(img, "lab")
        cen = _video_centres(c, before).double()
    else:
        planes = _planes64(_image(c["w"], c["h"], c["sigma"], _gen(seed)), c.get("color", "lab"))
        cen = _seeds64(planes, S, c.get("perturb", True))
    if kind == "warm":
        labels, votes = _warm_labels64(planes, _net_params(S, _gen(seed, 1)).double(), S, c["confidence"])
    else:
        (labels, dist), votes = _associate64(planes, S, wgt, cen, squared), None
    for i in range(c["iters"]):
        new = _means64(planes, labels, cen, votes if i == 0 else None)
        shift = float((new - cen).abs().sum()) / len(cen)
        cen = new
        labels, dist = _associate64(planes, S, wgt, cen, squared)
        if kind == "context" and shift < c["threshold"]:
            break
    energy = (dist.sqrt() if squared else dist).mean().reshape(1)
    if kind == "video":
        return dict(labels=None, centres=cen, counts=None)
    if kind == "context":
        return dict(rounds=None, energy=energy, labels=None, centres=cen, counts=None)
    out = dict(labels=None)
    if c.get("centres"):
        out["centres"] = cen
    if c.get("energy"):
        out["energy"] = energy
    if c["enforce"]:
        out["n_segments"] = None
    return out
