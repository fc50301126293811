"""The rendering backend's work as a client of this framework has it done,
each case one call (or one burst of calls) through the public entry points:
single frames from thumbnails to 4K, the batched and the serving form, the
allocation-free render and the JPEG payload.

`listed()` names the cases, `draw(rng)` gives another case of the same ranges,
`prepare` / `run` build and make one pass, `work` states the bytes and
operations a pass cannot do without, and `exact` gives the frame in 64 bits
where a frame leaves as floats.
"""
import math

import numpy as np
import torch

from paper_2605_08699_amd import synth, tigas

RUNGS = (0.25, 0.5, 0.75, 1.0)          # the resolution ladder of a request
LADDER_QUALITY = {0.25: 10, 0.5: 35, 0.75: 65, 1.0: 90}  # and its JPEG qualities


def _frame(name, n, w, h, scene="clusters", storage="f32", fmt="rgb8", degree=3, tiled=True, **kw):
    return dict(name=name, kind="frame", n=n, width=w, height=h, scene=scene, storage=storage, fmt=fmt,
                degree=degree, tiled=tiled, **kw)


def listed():
    return [
        # the smallest ordinary call: a 20k-Gaussian object in a thumbnail, tile chosen by the library
        _frame("frame_20k_256", 20_000, 256, 256, scene="uniform", tiled=False),
        # a ragged little frame at SH degree 0 (the backend's default quality), kept as floats
        _frame("frame_8k_333x217_floats", 8_000, 333, 217, scene="uniform", fmt="f32", degree=0),
        # a room-sized model at the top of the adaptive ladder, tile chosen by the library
        _frame("frame_1m_720p", 1_000_000, 1280, 720, tiled=False),
        # the headline workload: a 3M-Gaussian model at full HD
        _frame("frame_3m_1080p", 3_000_000, 1920, 1080),
        # the same from the half-precision storage that the serving form keeps resident
        _frame("frame_3m_1080p_f16", 3_000_000, 1920, 1080, storage="f16"),
        # a 4K frame: more tiles than a full-HD view, half-precision (bfloat16) model
        _frame("frame_3m_2160p_bf16", 3_000_000, 3840, 2160, storage="bf16"),
        # many clients' views of one model at the four ladder rungs in one call
        dict(name="batch_32_views_3m", kind="batch", n=3_000_000, views=32, width=1920, height=1080, storage="f16"),
        # a caller that may not allocate (captured or embedded in another pipeline)
        dict(name="noalloc_100k_540p", kind="noalloc", n=100_000, width=960, height=540, storage="f32"),
        # the server under a burst of clients: mixed models, rungs and JPEG payloads
        dict(name="serve_8_requests", kind="serve", n=300_000, n2=1_000_000, requests=8, width=1920, height=1080,
             storage="f16"),
        # the payload of one frame: the lowest and the highest rung of the ladder ...
        dict(name="jpeg_320x180_q10", kind="jpeg", width=320, height=180, quality=10),
        dict(name="jpeg_1280x720_q90", kind="jpeg", width=1280, height=720, quality=90),
        # ... and a 4K frame of a size that is no multiple of the 8-pixel blocks
        dict(name="jpeg_3837x2157_q85", kind="jpeg", width=3837, height=2157, quality=85),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["frame", "frame", "frame", "frame", "batch", "noalloc", "serve", "jpeg", "jpeg"])
    storage = rng.choice(["f32", "f16", "bf16"])
    if kind == "frame":
        fmt = rng.choice(["rgb8", "rgb8", "f32"])
        small = fmt == "f32"
        w = _log(rng, 120, 420 if small else 3840)
        return dict(kind="frame", n=_log(rng, 2_000, 20_000 if small else 3_000_000), width=w,
                    height=max(16, int(w * rng.uniform(0.5, 1.0 if w < 2160 else 0.5625))),
                    scene="uniform" if small else rng.choice(["uniform", "clusters", "clusters"]), storage=storage,
                    fmt=fmt, degree=rng.choice([0, 1, 2, 3, 3]), tiled=rng.random() < 0.7)
    if kind == "batch":
        w = _log(rng, 320, 1920)
        return dict(kind="batch", n=_log(rng, 20_000, 1_500_000), views=rng.randint(2, 24), width=w,
                    height=int(w * rng.uniform(0.5, 0.75)), storage=storage)
    if kind == "noalloc":
        w = _log(rng, 160, 1280)
        return dict(kind="noalloc", n=_log(rng, 2_000, 150_000), width=w, height=int(w * rng.uniform(0.5, 0.75)),
                    storage=storage)
    if kind == "serve":
        return dict(kind="serve", n=_log(rng, 20_000, 400_000), n2=_log(rng, 100_000, 1_000_000),
                    requests=rng.randint(1, 16), width=1920, height=1080, storage=rng.choice(["f16", "bf16"]))
    w = _log(rng, 64, 3840)
    return dict(kind="jpeg", width=w, height=max(8, int(w * rng.uniform(0.5, 1.0 if w < 2160 else 0.5625))),
                quality=rng.choice([10, 35, 65, 90, rng.randint(1, 100)]))


# ------------------------------------------------------------------ inputs

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _gen(seed):
    return torch.Generator(device=_device()).manual_seed(int(seed))


def _scene(kind, n, seed, degree=3):
    """A synthetic model with the attribute distributions of synth.py: centres
    uniform in a box, or 60 % in anisotropic clusters and 40 % flattened
    splats on the clusters' shells."""
    dev, g = _device(), _gen(seed)
    rn = lambda *s: torch.randn(*s, generator=g, device=dev)
    ls = rn(n, 3) * 0.5 - 4.0
    q = rn(n, 4)
    q = q / q.norm(dim=1, keepdim=True)
    logit = rn(n) * 1.5
    sh = torch.zeros(n, 16, 3, device=dev)
    nc = (degree + 1) ** 2
    sh[:, :nc] = rn(n, nc, 3) * 0.05
    sh[:, 0] *= 10.0
    if kind == "uniform":
        mu = torch.rand(n, 3, generator=g, device=dev) * 2.0 - 1.0
    else:
        m = 64
        centre = torch.rand(m, 3, generator=g, device=dev) * 10.0 - 5.0
        sig = torch.rand(m, 3, generator=g, device=dev) * 1.3 + 0.2
        axes = torch.linalg.qr(rn(m, 3, 3).cpu())[0].to(dev)
        k = torch.randint(0, m, (n,), generator=g, device=dev)
        xi = rn(n, 3)
        shell = torch.rand(n, generator=g, device=dev) < 0.4
        xi = torch.where(shell[:, None], 2.0 * xi / xi.norm(dim=1, keepdim=True), xi)
        mu = centre[k] + (axes[k] * (sig[k] * xi)[:, None, :]).sum(2)
        mu = torch.remainder(mu + 5.0, 10.0) - 5.0
        ls[:, 2] = torch.where(shell, rn(n) * 0.3 - 7.0, ls[:, 2])
    host = lambda t: t.cpu().numpy()
    return synth.Scene(host(mu), host(ls), host(q), host(logit), host(sh), degree)


def _poses(seed, count, radius):
    """Poses of a client's walk that starts on a sphere around the model, looking at it."""
    r = np.random.default_rng([int(seed) & 0xffffffff, 77])
    start = r.normal(size=3)
    start[2] = -abs(start[2]) - 0.5
    start *= radius / np.linalg.norm(start)
    return synth.trajectory(seed=int(seed) & 0xffffffff, n_poses=count, t0=start, R0=synth.look_at(start))


def _image(w, h, seed):
    """An RGB8 frame with the statistics of a rendered view: smooth shading,
    soft blobs, some fine texture."""
    dev, g = _device(), _gen(seed)
    img = torch.full((1, 3, h, w), 0.4, device=dev)
    for cells, amp in ((3, 0.30), (9, 0.20), (30, 0.12), (90, 0.07), (240, 0.04)):
        gh, gw = min(h, max(2, cells * h // max(w, h) + 2)), min(w, max(2, cells * w // max(w, h) + 2))
        f = torch.randn(1, 3, gh, gw, generator=g, device=dev) * 0.4 + torch.randn(1, 1, gh, gw, generator=g, device=dev)
        img += amp * torch.nn.functional.interpolate(f, size=(h, w), mode="bilinear", align_corners=True)
    img += 0.008 * torch.randn(1, 3, h, w, generator=g, device=dev)
    return (img[0].clamp(0, 1) * 255.0 + 0.5).to(torch.uint8).permute(1, 2, 0).contiguous()


class _Held:
    """A context with what one program keeps in it, given back with the state."""

    def __init__(self):
        self.ctx = tigas.Context(0)
        self.server = None

    def __del__(self):
        if self.server is not None:
            self.server.close()
        self.ctx.close()


_noalloc_stream = []  # the entry point's calls on one device may not overlap: one stream for all of them


def _out(w, h, fmt="rgb8"):
    return torch.empty((h, w, 3), dtype=torch.uint8 if fmt == "rgb8" else torch.float32, device="cuda")


def prepare(case, seed):
    held = _Held()
    st = dict(held=held, kind=case["kind"])
    w, h = case["width"], case["height"]
    if case["kind"] == "jpeg":
        st.update(rgb=_image(w, h, seed), quality=case["quality"])
        # a program that sends frames keeps one payload buffer: as large as the raw frame and header
        st["out"] = torch.zeros(w * h * 3 + 4096, dtype=torch.uint8, device="cuda")
        return st
    radius = 3.0 if case.get("scene") == "uniform" else 8.0
    scene = _scene(case.get("scene", "clusters"), case["n"], seed, case.get("degree", 3))
    k = synth.fov_intrinsics(w, h)
    st["scene"] = held.ctx.load_scene(scene, storage=case["storage"])
    if case["kind"] == "frame":
        fmt = case["fmt"]
        st.update(pose=_poses(seed, 1, radius)[0], k=k, w=w, h=h, out=_out(w, h, fmt),
                  opt=dict(fmt=fmt, bg=(0.1, 0.2, 0.3) if fmt == "f32" else (0.0, 0.0, 0.0)))
        if case["tiled"]:
            st["opt"].update(tile=(16, 32), batch_depth=64)  # what the serving form asks for
    elif case["kind"] == "noalloc":
        if not _noalloc_stream:
            _noalloc_stream.append(torch.cuda.Stream())
        st.update(pose=_poses(seed, 1, radius)[0], k=k, w=w, h=h, out=_out(w, h), stream=_noalloc_stream[0],
                  counters=torch.zeros(6, dtype=torch.int32, device="cuda"))
    elif case["kind"] == "batch":
        v = case["views"]
        st["scales"] = [RUNGS[i % 4] for i in range(v)]
        st["poses"] = _poses(seed, 9 * v, radius)[::9]
        st.update(ks=[k] * v, ws=[w] * v, hs=[h] * v, scenes=[st["scene"]] * v)
        st["outs"] = [_out(*tigas.output_size(w, h, s)) for s in st["scales"]]
    else:
        second = held.ctx.load_scene(_scene("clusters", case["n2"], seed + 1), storage=case["storage"])
        held.server = tigas.Server(held.ctx, slots=2, max_batch=64, max_batch_pixels=6_000_000)
        st.update(reqs=[], frames=[], payloads=[])
        for i in range(case["requests"]):
            s = RUNGS[(i * 3 + 1) % 4]
            ow, oh = tigas.output_size(w, h, s)
            st["frames"].append(_out(ow, oh))
            st["payloads"].append(torch.zeros(ow * oh * 3 + 4096, dtype=torch.uint8, device="cuda"))
            st["reqs"].append(tigas.request_c(st["scene"] if i % 2 else second, _poses(seed + 10 + i, 1, radius)[0], k,
                                              w, h, st["frames"][i], client=i, res_scale=s,
                                              jpeg_quality=LADDER_QUALITY[s], jpeg_out=st["payloads"][i]))
    torch.cuda.synchronize()
    return st


def run(st):
    ctx = st["held"].ctx
    if st["kind"] == "frame":
        return ctx.render(st["scene"], st["pose"], st["k"], st["w"], st["h"], out=st["out"], **st["opt"])
    if st["kind"] == "noalloc":
        ctx.render_noalloc(st["scene"], st["pose"], st["k"], st["w"], st["h"], st["out"], counters=st["counters"],
                           stream=st["stream"].cuda_stream)
        return st["out"]
    if st["kind"] == "batch":
        return ctx.render_batch(st["scenes"], st["poses"], st["ks"], st["ws"], st["hs"], res_scales=st["scales"],
                                tile=(16, 32), batch_depth=64, outs=st["outs"])
    if st["kind"] == "jpeg":
        out, n = ctx.jpeg_encode(st["rgb"], st["quality"], out=st["out"])
        return out, n
    server = st["held"].server
    first = server.submit(st["reqs"][0])
    for r in st["reqs"][1:]:
        server.submit(r)
    server.drain()
    size = {c["id"] - first: c["jpeg_bytes"] for c in server.poll()}
    return [(f, p, size[i]) for i, (f, p) in enumerate(zip(st["frames"], st["payloads"]))]


# -------------------------------------------------------- what a pass needs

def _frame_work(n, w, h, storage="f32", fmt="rgb8", degree=3):
    # every Gaussian's centre and shape, the colour of the half a view holds,
    # the frame; some 300 operations to project a Gaussian, and along a pixel's
    # ray the composited layers (21 operations each) until it is opaque
    el = 4 if storage == "f32" else 2
    nbytes = n * (12 + 8 * el) + n * 0.5 * 3 * (degree + 1) ** 2 * el + w * h * 3 * (1 if fmt == "rgb8" else 4)
    return nbytes, n * 300.0 + w * h * 21.0 * min(40.0, n / 300.0)


def work(case):
    w, h = case["width"], case["height"]
    if case["kind"] == "jpeg":
        # the frame read once, about a tenth of it written; 2 x 512 FMAs and the
        # colour transform per 8x8 block of each component
        return dict(bytes=w * h * 3 * 1.1, flops=w * h * 3 * 40.0)
    if case["kind"] in ("frame", "noalloc"):
        b, f = _frame_work(case["n"], w, h, case["storage"], case.get("fmt", "rgb8"), case.get("degree", 3))
        return dict(bytes=b, flops=f)
    total = dict(bytes=0.0, flops=0.0)
    for i in range(case["views"] if case["kind"] == "batch" else case["requests"]):
        s = RUNGS[i % 4] if case["kind"] == "batch" else RUNGS[(i * 3 + 1) % 4]
        ow, oh = tigas.output_size(w, h, s)
        n = case["n"] if case["kind"] == "batch" or i % 2 else case["n2"]
        # a batch reads its model once for all views
        b, f = _frame_work(n if case["kind"] == "serve" or i == 0 else 0, ow, oh, case["storage"])
        total["bytes"] += b + (ow * oh * 0.3 if case["kind"] == "serve" else 0.0)
        total["flops"] += f + (n * 300.0 if case["kind"] == "batch" and i else 0.0)
    return total


# ------------------------------------------------------------- in 64 bits

def _f32(x):
    return x.to(torch.float32).to(torch.float64)


def _sh_basis(d):
    x, y, z = d[:, 0], d[:, 1], d[:, 2]
    p = math.pi
    c0, c1 = 0.5 * math.sqrt(1 / p), math.sqrt(3 / (4 * p))
    c2, c3 = 0.5 * math.sqrt(15 / p), 0.25 * math.sqrt(5 / p)
    a, b = 0.25 * math.sqrt(35 / (2 * p)), 0.5 * math.sqrt(105 / p)
    c, e = 0.25 * math.sqrt(21 / (2 * p)), 0.25 * math.sqrt(7 / p)
    one = torch.ones_like(x)
    return torch.stack([
        c0 * one, -c1 * y, c1 * z, -c1 * x,
        c2 * x * y, -c2 * y * z, c3 * (3 * z * z - 1), -c2 * x * z, 0.5 * c2 * (x * x - y * y),
        -a * y * (3 * x * x - y * y), b * x * y * z, -c * y * (5 * z * z - 1), e * z * (5 * z * z - 3),
        -c * x * (5 * z * z - 1), 0.5 * b * z * (x * x - y * y), -a * x * (x * x - 3 * y * y)], 1)


def exact(case, seed):
    """The float frames: every Gaussian at every pixel, front to back."""
    if case["kind"] != "frame" or case["fmt"] != "f32":
        return None  # bytes
    dev, w, h = _device(), case["width"], case["height"]
    scene = _scene(case["scene"], case["n"], seed, case["degree"])
    pose = _poses(seed, 1, 3.0 if case["scene"] == "uniform" else 8.0)[0]
    k = synth.fov_intrinsics(w, h)
    half = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[case["storage"]]
    t64 = lambda a: torch.as_tensor(np.asarray(a), device=dev).to(torch.float64)
    kept = lambda a: torch.as_tensor(np.asarray(a), device=dev).to(half).to(torch.float64)
    mu, ls, q = t64(scene.means), kept(scene.log_scales), kept(scene.quats)
    op, sh = torch.sigmoid(kept(scene.opacity_logits)), kept(scene.sh)
    R, t = t64(pose.R), t64(pose.t)
    V = R.T
    # the order key is defined in 32 bits: nested fused multiply-adds
    z = _f32(mu[:, 2] * V[2, 2] + _f32(-(V[2] * t).sum()))
    z = _f32(mu[:, 1] * V[2, 1] + z)
    z = _f32(mu[:, 0] * V[2, 0] + z)
    keep = torch.nonzero((z > float(np.float32(0.2))) & (q.norm(dim=1) > 0))[:, 0]
    keep = keep[torch.sort(z[keep], stable=True)[1]]
    mu, ls, op, sh = mu[keep], ls[keep], op[keep], sh[keep]
    q = q[keep] / q[keep].norm(dim=1, keepdim=True)
    a, b, c, d = q.unbind(1)
    rot = torch.stack([1 - 2 * (c * c + d * d), 2 * (b * c - a * d), 2 * (b * d + a * c),
                       2 * (b * c + a * d), 1 - 2 * (b * b + d * d), 2 * (c * d - a * b),
                       2 * (b * d - a * c), 2 * (c * d + a * b), 1 - 2 * (b * b + c * c)], 1).reshape(-1, 3, 3)
    m = rot * torch.exp(ls)[:, None, :]
    view = mu - t
    p = (V[None] * view[:, None, :]).sum(2)
    fx, fy, cx, cy = (float(np.float32(v)) for v in (k.fx, k.fy, k.cx, k.cy))
    u, v = fx * p[:, 0] / p[:, 2] + cx, fy * p[:, 1] / p[:, 2] + cy
    lx, ly = 1.3 * max(cx, w - cx) / fx, 1.3 * max(cy, h - cy) / fy
    rx, ry = (p[:, 0] / p[:, 2]).clamp(-lx, lx), (p[:, 1] / p[:, 2]).clamp(-ly, ly)
    j0 = (fx / p[:, 2])[:, None] * (V[0] - rx[:, None] * V[2])
    j1 = (fy / p[:, 2])[:, None] * (V[1] - ry[:, None] * V[2])
    m0, m1 = (j0[:, :, None] * m).sum(1), (j1[:, :, None] * m).sum(1)
    s00, s01, s11 = (m0 * m0).sum(1) + float(np.float32(0.3)), (m0 * m1).sum(1), (m1 * m1).sum(1) + float(np.float32(0.3))
    det = s00 * s11 - s01 * s01
    basis = _sh_basis(view / view.norm(dim=1, keepdim=True))[:, :(case["degree"] + 1) ** 2]
    rgb = (0.5 + (basis[:, :, None] * sh[:, :basis.shape[1]]).sum(1)).clamp_min(0)
    a_min, a_max, t_min = (float(np.float32(x)) for x in (1 / 255, 0.99, 1e-4))
    bg = torch.tensor([0.1, 0.2, 0.3], device=dev).to(torch.float64)
    px = torch.arange(w, device=dev).to(torch.float64) + 0.5
    img = torch.zeros(h, w, 3, dtype=torch.float64, device=dev)
    rows = max(1, 16384 // w)
    for y0 in range(0, h, rows):
        y = torch.arange(y0, min(h, y0 + rows), device=dev).to(torch.float64) + 0.5
        gx, gy = px.repeat(len(y)), y.repeat_interleave(w)
        T = torch.ones(len(gx), dtype=torch.float64, device=dev)
        done = torch.zeros(len(gx), dtype=torch.bool, device=dev)
        col = torch.zeros(len(gx), 3, dtype=torch.float64, device=dev)
        for g in range(0, len(keep), 512):
            s = slice(g, g + 512)
            dx, dy = gx[:, None] - u[s], gy[:, None] - v[s]
            e = (s11[s] * dx * dx - 2 * s01[s] * dx * dy + s00[s] * dy * dy) / det[s]
            al = (op[s] * torch.exp(-0.5 * e)).clamp(max=a_max)
            al = torch.where(al >= a_min, al, 0.0)
            after = T[:, None] * torch.cumprod(1 - al, 1)
            before = torch.cat([T[:, None], after[:, :-1]], 1)
            on = (after >= t_min) & ~done[:, None]
            wgt = torch.where(on, al * before, 0.0)
            col += (wgt[:, :, None] * rgb[s]).sum(1)
            T = torch.where(on, after, 1.0).amin(1).minimum(T)
            done |= ~on[:, -1]
        img[y0:y0 + len(y)] = (col + T[:, None] * bg).reshape(len(y), w, 3)
    return img
