"""Parity of the GPU JPEG encoder with the JPEG oracle (needs an MI355X): the
streams must be byte-identical.  Every call goes through the C ABI."""
import io
import math

import numpy as np
import pytest
import torch
from PIL import Image

from oracle import jpeg as oj
from paper_2605_08699_amd import synth, tigas

pytestmark = pytest.mark.gpu

LADDER = ((320, 180, 10), (640, 360, 35), (960, 540, 65), (1280, 720, 90))  # Table 1 rungs


@pytest.fixture(scope="module")
def ctx():
    c = tigas.Context(0)
    yield c
    c.close()


def _say(*a):
    print(*a, flush=True)


def _image(H, W, seed):
    rng = np.random.default_rng(seed)
    y, x = np.mgrid[0:H, 0:W]
    img = np.stack([128 + 110 * np.sin(x / 5.0 + y / 9.0), 128 + 100 * np.cos(y / 4.0 - x / 13.0),
                    (x * 5 + y * 3) % 256], -1)
    img = img + rng.normal(0, 10, img.shape)
    img[: max(1, H // 5)] = 255  # saturated rows: 0xFF bytes in the coded data
    return np.clip(np.rint(img), 0, 255).astype(np.uint8)


def _gpu(img):
    return torch.from_numpy(np.ascontiguousarray(img)).cuda()


@pytest.mark.parametrize("size", [(1, 1), (8, 8), (13, 37), (72, 120), (181, 323)])
@pytest.mark.parametrize("q", [1, 10, 35, 65, 90, 100])
def test_stream_equals_oracle(ctx, size, q):
    H, W = size
    img = _image(H, W, seed=H * 7 + W + q)
    _say("jpeg", size, q)
    got = ctx.jpeg_bytes(_gpu(img), q)
    want = oj.encode(img, q)
    assert len(got) == len(want)
    assert got == want


@pytest.mark.parametrize("mcus", [39, 40, 41, 79, 81])
def test_interval_edges(ctx, mcus):
    # one restart interval is 40 MCUs: the last one short, full, and a single
    # MCU over, with the last column of pixels inside a block
    img = _image(7, mcus * 8 - 3, seed=mcus)
    _say("jpeg interval", mcus)
    for q in (35, 90):
        assert ctx.jpeg_bytes(_gpu(img), q) == oj.encode(img, q)


@pytest.mark.parametrize("kind", ["noise", "two_level", "sparse", "flat"])
def test_interval_bit_counts(ctx, kind):
    # from one code per block to intervals of more bits than one window of
    # the bit stream holds (65536); single high-frequency values follow runs of
    # zeros of every length
    rng = np.random.default_rng(17)
    H, W = 24, 328
    if kind == "noise":
        img = rng.integers(0, 256, (H, W, 3)).astype(np.uint8)
    elif kind == "two_level":
        img = (rng.integers(0, 2, (H, W, 3)) * 255).astype(np.uint8)
    elif kind == "flat":
        img = np.full((H, W, 3), 77, np.uint8)
    else:
        y, x = np.mgrid[0:H, 0:W]
        u, v = (x // 8) % 8, (x // 64 + y // 8) % 8  # one DCT basis function per block
        img = 128 + 60 * np.cos((2 * (x % 8) + 1) * u * np.pi / 16) * np.cos((2 * (y % 8) + 1) * v * np.pi / 16)
        img = np.repeat(np.rint(img)[:, :, None], 3, 2).astype(np.uint8)
    for q in (10, 90, 100):
        _say("jpeg bits", kind, q)
        want = oj.encode(img, q)
        if kind == "two_level" and q == 100:
            assert len(want) > 3 * 65536 // 8
        assert ctx.jpeg_bytes(_gpu(img), q) == want


def test_many_payloads_in_one_batch(ctx):
    # more payloads than one pair of launches takes, of different sizes and
    # qualities: each is its own frame's stream
    scene, poses, _, _, _ = synth.c1_single_view()
    s = ctx.load_scene(scene)
    k = synth.fov_intrinsics(200, 120)
    frames, outs, reqs = [], [], []
    with tigas.Server(ctx, slots=1) as sv:
        for i in range(37):
            sc = (0.25, 0.5, 0.75, 1.0)[i % 4]
            ow, oh = tigas.output_size(200, 120, sc)
            frames.append(torch.empty((oh, ow, 3), dtype=torch.uint8, device="cuda"))
            outs.append(torch.zeros(1 << 16, dtype=torch.uint8, device="cuda"))
            reqs.append(tigas.request_c(s, poses[0], k, 200, 120, frames[i], client=i, res_scale=sc,
                                        jpeg_quality=10 + 2 * i, jpeg_out=outs[i]))
        for r in reqs:
            sv.submit(r)
        sv.drain()
        done = {c["id"]: c for c in sv.poll()}
    assert max(c["batch_size"] for c in done.values()) > 16
    for i in range(37):
        want = oj.encode(frames[i].cpu().numpy(), 10 + 2 * i)
        assert done[i]["status"] == 0 and done[i]["jpeg_bytes"] == len(want)
        assert bytes(outs[i][:len(want)].cpu().numpy()) == want
    s.free()


def test_wide_frames_and_repeated_calls(ctx):
    # wide frames (intervals wrap across MCU rows), then a smaller frame on the
    # same buffers, then the large one again: the interval bit buffers must
    # come back cleared
    for H, W, q in ((24, 4096, 90), (16, 40, 35), (24, 4096, 90), (1, 6000, 100), (300, 9, 65)):
        img = _image(H, W, seed=W + H)
        _say("jpeg", (H, W), q)
        assert ctx.jpeg_bytes(_gpu(img), q) == oj.encode(img, q)


def test_rendered_ladder_frames(ctx):
    # frames the rasterizer renders at the ladder's resolutions, encoded at
    # the ladder's quality factors
    scene, poses, _, _, _ = synth.c1_single_view()
    s = ctx.load_scene(scene)
    for w, h, q in LADDER:
        kk = synth.fov_intrinsics(w, h)
        frame = torch.empty((h, w, 3), dtype=torch.uint8, device="cuda")
        ctx.render(s, poses[0], kk, w, h, out=frame)
        _say("jpeg ladder", (w, h), q)
        got = ctx.jpeg_bytes(frame, q)
        img = frame.cpu().numpy()
        assert got == oj.encode(img, q)
        dec = np.asarray(Image.open(io.BytesIO(got)).convert("RGB")).astype(np.float64)
        mse = ((dec - img) ** 2).mean()
        assert 10 * math.log10(255.0 ** 2 / max(mse, 1e-12)) > {10: 25.0, 35: 30.0, 65: 33.0, 90: 38.0}[q]
    s.free()


def test_small_buffer_reports_the_length(ctx):
    img = _image(40, 64, seed=3)
    t = _gpu(img)
    want = oj.encode(img, 90)
    small = torch.zeros(100, dtype=torch.uint8, device="cuda")
    with pytest.raises(tigas.TigasError) as e:
        ctx.jpeg_encode(t, 90, out=small)
    assert "smaller" in str(e.value)
    assert bytes(small.cpu().numpy()) == want[:100]
    out, n = ctx.jpeg_encode(t, 90)
    assert n == len(want) and bytes(out[:n].cpu().numpy()) == want


def test_invalid_arguments(ctx):
    img = _gpu(_image(8, 8, seed=1))
    for q in (0, 101):
        with pytest.raises(tigas.TigasError):
            ctx.jpeg_encode(img, q)
    wide = _gpu(np.zeros((1, 65536, 3), np.uint8))
    with pytest.raises(tigas.TigasError):
        ctx.jpeg_encode(wide, 90)
