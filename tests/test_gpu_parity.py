"""Parity of the HIP path with the FP64 oracle (needs an MI355X).

Every call goes through the C ABI of libtigas.so via the ctypes binding.
"""
import ctypes
import dataclasses
import math

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2605_08699_amd import synth, tigas
from tests import gpu_checks as gc
from tests.handmade import eye_pose, intr, make_scene, random_tiny_scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = tigas.Context(0)
    yield c
    c.close()


@pytest.fixture(scope="module")
def c1():
    return synth.c1_single_view()


def _say(*a):
    print(*a, flush=True)


def test_wave_scan_dpp():
    rng = np.random.default_rng(0)
    for n in (64, 200, 4096 + 17):
        x = rng.integers(0, 1000, n).astype(np.uint32)
        got = tigas.selftest_wave_scan(x)
        want = np.concatenate([np.cumsum(x[i:i + 64]) for i in range(0, n, 64)]).astype(np.uint32)
        np.testing.assert_array_equal(got, want)


def test_c1_preprocess_matches_oracle(ctx, c1):
    scene, poses, k, W, H = c1
    s = ctx.load_scene(scene)
    _say("c1 preprocess", scene.n, W, H)
    dbg = ctx.render_debug(s, poses[0], k, W, H)
    proj = orc.preprocess(scene, poses[0], k, W, H)
    err = gc.check_preprocess(dbg, proj, W, H)
    _say("k1 errors", err)
    assert err["uv"] < 1e-4


@pytest.mark.parametrize("binning", [True, False])
@pytest.mark.parametrize("tile", [(16, 16), (8, 8), (16, 32), (32, 16)])
def test_c1_tile_lists_sort_and_ranges_bit_exact(ctx, c1, tile, binning):
    """Both placements of the tile digit (counting, radix passes) give the
    sorted list of the plain 64-bit key sort."""
    scene, poses, k, W, H = c1
    s = ctx.load_scene(scene)
    _say("c1 tiles", tile, "binning", binning)
    ctx.set_tile_binning(binning)
    try:
        dbg = ctx.render_debug(s, poses[0], k, W, H, tile=tile)
        passes = ctx.stats()["sort_passes"]
    finally:
        ctx.set_tile_binning(True)
    gc.check_tiles(dbg, *tile)
    assert dbg["n_dup"] > scene.n
    # 3 depth passes, then one counting placement or the radix tile passes
    assert passes == (4 if binning else 3 + math.ceil(math.log2((W // tile[0]) * (H // tile[1])) / 8))


@pytest.mark.parametrize("binning", [True, False])
def test_c1_three_and_four_pass_depth_sorts_give_identical_lists_and_frames(ctx, c1, binning):
    scene, poses, k, W, H = c1
    s = ctx.load_scene(scene)
    got = {}
    ctx.set_tile_binning(binning)
    try:
        for passes in (3, 4):
            ctx.set_depth_passes(passes)
            dbg = ctx.render_debug(s, poses[0], k, W, H, tile=(16, 16))
            got[passes] = (dbg, ctx.stats())
    finally:
        ctx.set_depth_passes(3)
        ctx.set_tile_binning(True)
    _say("depth passes", {p: g[1]["sort_passes"] for p, g in got.items()})
    tile_passes = 1 if binning else math.ceil(math.log2((W // 16) * (H // 16)) / 8)
    for passes, (dbg, st) in got.items():
        gc.check_tiles(dbg, 16, 16)
        assert st["rerenders"] == 0
        assert st["sort_passes"] == passes + tile_passes
    for key in ("svals", "skeys", "ranges", "image"):
        np.testing.assert_array_equal(got[3][0][key], got[4][0][key])


def test_depth_passes_other_than_three_or_four_are_refused(ctx):
    for bad in (0, 2, 5, -1):
        with pytest.raises(tigas.TigasError, match="E_INVALID"):
            ctx.set_depth_passes(bad)
    ctx.set_depth_passes(3)


def test_frame_too_deep_for_three_passes_is_rendered_again_with_four():
    # depths from 0.5 to 2e7 (their FP32 keys span more than 2^27), sizes
    # growing with depth so that every Gaussian covers a few pixels
    rng = np.random.default_rng(5)
    n = 600
    z = np.exp(rng.uniform(math.log(0.5), math.log(2e7), n))
    means = np.column_stack([rng.uniform(-0.35, 0.35, n) * z, rng.uniform(-0.25, 0.25, n) * z, z])
    ls = np.repeat(np.log(0.02 * z)[:, None], 3, axis=1) + rng.normal(0.0, 0.3, (n, 3))
    scene = make_scene(means, ls, rng.normal(size=(n, 4)), rng.normal(1.0, 1.0, n), rng.uniform(0.0, 1.0, (n, 3)))
    W, H = 200, 136
    k = intr(150.0, W / 2, H / 2)
    c = tigas.Context(0)  # the switch to four passes is kept per context
    try:
        s = c.load_scene(scene)
        img = c.render(s, eye_pose(), k, W, H, fmt="f32", tile=(16, 16))
        st = c.stats()
        _say("deep frame", st)
        assert st["rerenders"] == 1 and st["sort_passes"] == 5
        proj = orc.preprocess(scene, eye_pose(), k, W, H)
        br, nb = orc.render_frame(proj)
        res = gc.check_frame_pixels(img.reshape(-1, 3), br.reshape(-1, br.shape[2], 4), nb.reshape(-1))
        assert res["n_bad"] == 0 and res["n_unresolved"] == 0, res
        # later frames take four passes from the start
        dbg = c.render_debug(s, eye_pose(), k, W, H, tile=(16, 16))
        st2 = c.stats()
        assert st2["rerenders"] == 0 and st2["sort_passes"] == 5
        zk = dbg["zkey"][dbg["touched"] > 0].astype(np.int64)
        assert zk.max() - (zk.min() & ~511) >= 1 << 27  # the frame is too deep for three passes
        gc.check_tiles(dbg, 16, 16)
        np.testing.assert_array_equal(img, dbg["image"])
    finally:
        c.close()


def test_frame_just_shallow_enough_keeps_three_passes(ctx):
    # the same construction with depths from 0.5 to 1000: keys span less than 2^27
    rng = np.random.default_rng(6)
    n = 600
    z = np.exp(rng.uniform(math.log(0.5), math.log(1000.0), n))
    means = np.column_stack([rng.uniform(-0.35, 0.35, n) * z, rng.uniform(-0.25, 0.25, n) * z, z])
    ls = np.repeat(np.log(0.02 * z)[:, None], 3, axis=1)
    scene = make_scene(means, ls, None, np.full(n, 1.0), rng.uniform(0.0, 1.0, (n, 3)))
    W, H = 200, 136
    k = intr(150.0, W / 2, H / 2)
    s = ctx.load_scene(scene)
    dbg = ctx.render_debug(s, eye_pose(), k, W, H, tile=(16, 16))
    st = ctx.stats()
    zk = dbg["zkey"][dbg["touched"] > 0].astype(np.int64)
    assert 1 << 25 < zk.max() - (zk.min() & ~511) < 1 << 27
    assert st["rerenders"] == 0 and st["sort_passes"] == 4
    gc.check_tiles(dbg, 16, 16)


def _depth_scene(kind, n):
    """n small Gaussians in view whose depths are spread in a way that the
    buckets of the depth sort meet in different forms."""
    rng = np.random.default_rng(n)
    if kind == "spread":
        z = rng.uniform(1.0, 9.0, n)
    elif kind == "equal":
        z = np.full(n, 4.0)
    elif kind == "two":
        z = np.where(rng.random(n) < 0.5, 3.0, 5.0)
    elif kind == "lattice":
        z = 2.0 + rng.integers(0, 40, n) * 0.125
    elif kind == "thin":  # a thin slab and one far Gaussian
        z = 5.0 + rng.normal(0.0, 1e-4, n)
        z[n // 2] = 900.0
    else:  # steps: half of them at one depth, the rest spread
        z = np.where(rng.random(n) < 0.5, 4.0, rng.uniform(1.0, 9.0, n))
    means = np.column_stack([rng.uniform(-0.3, 0.3, n) * z, rng.uniform(-0.2, 0.2, n) * z, z])
    ls = np.repeat(np.log(0.004 * z)[:, None], 3, axis=1)
    return make_scene(means, ls, None, rng.normal(0.0, 1.0, n), rng.uniform(0.0, 1.0, (n, 3)))


@pytest.mark.parametrize("kind,n", [("spread", n) for n in (1, 63, 65, 257, 2047, 2049, 4096, 4097, 8193, 70_001)] +
                         [(k, n) for k in ("equal", "two", "lattice", "thin", "steps") for n in (3000, 60_000)])
def test_depth_buckets_give_the_stable_order(ctx, kind, n):
    """Segments and buckets of every fill, equal depths (more than a bucket's
    workgroup holds at once, too) and a depth range that one far Gaussian
    stretches: the lists of the plain 64-bit key sort, and the frame of the
    four-pass radix sort."""
    scene = _depth_scene(kind, n)
    W, H = 160, 112
    k = intr(150.0, W / 2, H / 2)
    s = ctx.load_scene(scene)
    _say("depth buckets", kind, n)
    dbg = ctx.render_debug(s, eye_pose(), k, W, H, tile=(16, 16))
    assert ctx.stats()["rerenders"] == 0 and dbg["n_dup"] > 0
    gc.check_tiles(dbg, 16, 16)
    ctx.set_depth_passes(4)
    try:
        ref = ctx.render(s, eye_pose(), k, W, H, fmt="f32", tile=(16, 16))
    finally:
        ctx.set_depth_passes(3)
    np.testing.assert_array_equal(dbg["image"], ref)
    s.free()


@pytest.mark.parametrize("kind,n", [("equal", 17_000), ("equal", 200_000), ("steps", 200_000), ("slab", 66_000),
                                    ("slab", 200_000)])
def test_crowded_depth_buckets(ctx, kind, n):
    """More Gaussians at about one depth than a workgroup is given to sort: the
    frame is rendered again with the radix passes, once; the form without a
    second attempt sorts them in their bucket, to the same frame."""
    import torch
    scene = _depth_scene("thin" if kind == "slab" else kind, n)
    if kind == "slab":  # 99 % of them in a few buckets: at least 39 % in one
        scene.means[::97, 2] = 900.0
    W, H = 160, 112
    k = intr(150.0, W / 2, H / 2)
    s = ctx.load_scene(scene)
    _say("crowded buckets", kind, n)
    out = torch.zeros((H, W, 3), dtype=torch.float32, device="cuda")
    ctx.render_noalloc(s, eye_pose(), k, W, H, out, fmt="f32", tile=(16, 16))
    torch.cuda.synchronize()
    try:
        img = ctx.render(s, eye_pose(), k, W, H, fmt="f32", tile=(16, 16))
        assert img.any() and ctx.stats()["rerenders"] == 1
        ctx.set_depth_passes(4)
        ref = ctx.render(s, eye_pose(), k, W, H, fmt="f32", tile=(16, 16))
        radix = torch.zeros_like(out)
        ctx.render_noalloc(s, eye_pose(), k, W, H, radix, fmt="f32", tile=(16, 16))
        torch.cuda.synchronize()
    finally:
        ctx.set_depth_passes(3)
    np.testing.assert_array_equal(img, ref)
    np.testing.assert_array_equal(radix.cpu().numpy(), ref)
    np.testing.assert_array_equal(out.cpu().numpy(), ref)
    s.free()


def _noalloc_frame(ctx, s, k, W, H):
    import torch
    out = torch.zeros((H, W, 3), dtype=torch.float32, device="cuda")
    ctx.render_noalloc(s, eye_pose(), k, W, H, out, fmt="f32", tile=(16, 16))
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("kind,n", [("equal", n) for n in (2047, 2049, 4095, 4097, 8191, 16_385, 131_073, 300_000)] +
                         [(k, n) for k in ("two", "lattice", "thin", "steps") for n in (4097, 17_000, 200_000)])
def test_crowded_depths_are_parted_by_order_statistics(ctx, kind, n):
    """Depths that crowd, in the form that parts them on the spot: the frame of
    the four-pass radix sort."""
    scene = _depth_scene(kind, n)
    W, H = 160, 112
    k = intr(150.0, W / 2, H / 2)
    s = ctx.load_scene(scene)
    _say("parted by order statistics", kind, n)
    got = _noalloc_frame(ctx, s, k, W, H)
    ctx.set_depth_passes(4)
    try:
        want = ctx.render(s, eye_pose(), k, W, H, fmt="f32", tile=(16, 16))
    finally:
        ctx.set_depth_passes(3)
    assert want.any()
    np.testing.assert_array_equal(got, want)
    s.free()


def test_frame_of_one_depth_takes_about_as_long_as_any_other(ctx):
    """200k Gaussians of one depth, in the form without a second attempt: within
    four times the frame of as many at spread depths (in one bucket it was 18)."""
    import time

    import torch
    W, H, n = 960, 540, 200_000
    k = intr(480.0, W / 2, H / 2)
    out = torch.zeros((H, W, 3), dtype=torch.uint8, device="cuda")
    us = {}
    for kind in ("spread", "equal", "steps"):
        s = ctx.load_scene(_depth_scene(kind, n))
        times = []
        for _ in range(9):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(10):
                ctx.render_noalloc(s, eye_pose(), k, W, H, out, tile=(16, 16))
            torch.cuda.synchronize()
            times.append((time.perf_counter() - t0) * 1e5)
        us[kind] = sorted(times)[4]
        s.free()
    _say("us a frame", us)
    assert max(us["equal"], us["steps"]) < 4 * us["spread"]


def test_a_frame_that_needs_another_depth_order_changes_only_its_own_scene():
    """After a crowded frame and a too deep one, frames of other scenes, alone
    and in a batch with those, are in buckets and placed by counting as before;
    the two scenes' own next frames are rendered once; a new request for three
    passes starts afresh."""
    W, H = 160, 112
    k = intr(150.0, W / 2, H / 2)
    rng = np.random.default_rng(8)
    z = np.exp(rng.uniform(math.log(0.5), math.log(2e7), 600))
    deep = make_scene(np.column_stack([rng.uniform(-0.3, 0.3, 600) * z, rng.uniform(-0.2, 0.2, 600) * z, z]),
                      np.repeat(np.log(0.02 * z)[:, None], 3, axis=1), None, rng.normal(1.0, 1.0, 600),
                      rng.uniform(0.0, 1.0, (600, 3)))
    c = tigas.Context(0)

    def render(*scenes):
        n = len(scenes)
        out = c.render_batch(scenes, [eye_pose()] * n, [k] * n, [W] * n, [H] * n, fmt="f32", tile=(16, 16)) \
            if n > 1 else [c.render(scenes[0], eye_pose(), k, W, H, fmt="f32", tile=(16, 16))]
        st = c.stats()
        return out, (st["rerenders"], st["sort_passes"])

    try:
        plain, flat, far = (c.load_scene(x) for x in (_depth_scene("spread", 6000), _depth_scene("equal", 20_000), deep))
        own = {}
        for s, first, later in ((plain, (0, 4), (0, 4)), (flat, (1, 4), (0, 4)), (far, (1, 5), (0, 5))):
            (own[s],), how = render(s)
            assert how == first
            (again,), how = render(s)
            assert how == later
            np.testing.assert_array_equal(again, own[s])
        assert render(plain)[1] == (0, 4)
        for batch in ((plain, plain), (plain, flat), (flat, far, plain)):
            got, how = render(*batch)
            assert how == (0, 4), how
            for s, img in zip(batch, got):
                np.testing.assert_array_equal(img, own[s])
        c.set_depth_passes(4)
        for s in (plain, flat, far):
            (ref,), how = render(s)
            assert how == (0, 5)
            np.testing.assert_array_equal(ref, own[s])
        c.set_depth_passes(3)
        assert render(flat)[1] == (1, 4) and render(far)[1] == (1, 5) and render(plain)[1] == (0, 4)
    finally:
        c.close()


def test_switches_flipped_by_another_thread_change_no_frame():
    """The depth order, the placement and the culling switched by one thread
    while another renders single views and batches, crowded, deep and plain:
    every frame is the one of fixed switches."""
    import threading
    W, H = 700, 500
    k = intr(500.0, W / 2, H / 2)
    rng = np.random.default_rng(12)
    z = np.exp(rng.uniform(math.log(0.5), math.log(2e7), 600))
    deep = make_scene(np.column_stack([rng.uniform(-0.3, 0.3, 600) * z, rng.uniform(-0.2, 0.2, 600) * z, z]),
                      np.repeat(np.log(0.02 * z)[:, None], 3, axis=1), None, rng.normal(1.0, 1.0, 600),
                      rng.uniform(0.0, 1.0, (600, 3)))
    c = tigas.Context(0)
    try:
        ss = [c.load_scene(x) for x in (_depth_scene("spread", 6000), _depth_scene("equal", 20_000), deep)]
        want = [c.render(s, eye_pose(), k, W, H, fmt="f32", tile=(16, 16)) for s in ss]
        stop = threading.Event()

        def flip():
            i = 0
            while not stop.is_set():
                c.set_depth_passes(3 + i % 2)
                c.set_tile_binning(i % 3 != 0)
                c.set_tile_culling(i % 5 == 0)
                i += 1

        t = threading.Thread(target=flip)
        t.start()
        try:
            for i in range(150):
                if i % 3 == 2:
                    got = c.render_batch(ss, [eye_pose()] * 3, [k] * 3, [W] * 3, [H] * 3, fmt="f32", tile=(16, 16))
                else:
                    got = [c.render(s, eye_pose(), k, W, H, fmt="f32", tile=(16, 16)) for s in ss]
                for j in range(3):
                    np.testing.assert_array_equal(got[j], want[j], err_msg=f"pass {i}, scene {j}")
        finally:
            stop.set()
            t.join()
    finally:
        c.close()


@pytest.mark.parametrize("n,views", [(2_100_000, 1), (180_000, 48)])
def test_crowded_depths_of_large_plans(n, views):
    """Crowded depths in a view of 2048 buckets, of whose samples every second is
    sorted, and in 528 segments, which read the views' order statistics: the
    frames of the four-pass radix sort."""
    scene = _depth_scene("steps", n)
    W, H = (640, 400) if views == 1 else (66, 60)
    k = intr(600.0 if views == 1 else 40.0, W / 2, H / 2)
    poses = [eye_pose((0.01 * i, 0.0, -0.02 * i)) for i in range(views)]
    _say("crowded large plan", n, views)
    c = tigas.Context(0)
    try:
        s = c.load_scene(scene)
        for attempt in range(2):  # flagged and rendered again, then at once
            got = c.render_batch([s] * views, poses, [k] * views, [W] * views, [H] * views, fmt="f32", tile=(16, 16)) \
                if views > 1 else [c.render(s, poses[0], k, W, H, fmt="f32", tile=(16, 16))]
            st = c.stats()
            assert (st["rerenders"], st["sort_passes"]) == (1 - attempt, 4)
            if attempt == 0:
                first = got
        c.set_depth_passes(4)
        for i in (0, views // 2, views - 1):
            want = c.render(s, poses[i], k, W, H, fmt="f32", tile=(16, 16))
            assert want.any()
            np.testing.assert_array_equal(first[i], want)
            np.testing.assert_array_equal(got[i], want)
    finally:
        c.close()


@pytest.mark.parametrize("kind", ["equal", "deep"])
def test_batch_that_needs_another_depth_order_and_more_room(kind):
    """Views whose first attempt fits in shared lists but is rendered again
    with more entries than the first buffers hold (2^20): each frame is the
    view's own."""
    rng = np.random.default_rng(41)
    n, W, H = 30_000, 1920, 1080
    z = np.full(n, 4.0) if kind == "equal" else np.exp(rng.uniform(math.log(0.5), math.log(2e7), n))
    means = np.column_stack([rng.uniform(-0.9, 0.9, n) * z, rng.uniform(-0.5, 0.5, n) * z, z])
    scene = make_scene(means, np.repeat(np.log(0.0125 * z)[:, None], 3, axis=1), None, rng.normal(1.0, 0.3, n),
                       rng.uniform(0.0, 1.0, (n, 3)))
    k = intr(960.0, W / 2, H / 2)
    poses = [eye_pose(), eye_pose((0.05, 0.02, 0.0))]
    _say("batch rendered again", kind)
    c = tigas.Context(0)  # buffers and depth order of their own
    try:
        s = c.load_scene(scene)
        got = c.render_batch([s] * 2, poses, [k] * 2, [W] * 2, [H] * 2, fmt="f32", tile=(16, 16))
        st = c.stats()
        _say(st)
        assert st["duplicates"] > max(4 * 2 * n, 1 << 20)
        again = c.render_batch([s] * 2, poses, [k] * 2, [W] * 2, [H] * 2, fmt="f32", tile=(16, 16))
        assert c.stats()["rerenders"] == 0 and c.stats()["duplicates"] == st["duplicates"]
        c.set_depth_passes(4)
        for i in range(2):
            want = c.render(s, poses[i], k, W, H, fmt="f32", tile=(16, 16))
            assert want.any()
            np.testing.assert_array_equal(got[i], want)
            np.testing.assert_array_equal(again[i], want)
    finally:
        c.close()


def test_depth_buckets_of_several_views_and_a_culled_one(ctx):
    """Views of scenes of different sizes, one of which shows nothing, in one
    sequence: each frame is the view's own."""
    scenes = [ctx.load_scene(_depth_scene("spread", n)) for n in (70_000, 300, 5000)]
    poses = [eye_pose(), eye_pose(), synth.Pose(np.eye(3, dtype=np.float32), np.array([0, 0, 500.0], np.float32)),
             eye_pose()]
    which = [scenes[0], scenes[1], scenes[0], scenes[2]]
    sizes = [(160, 112), (64, 48), (160, 112), (33, 200)]
    ks = [intr(150.0, w / 2, h / 2) for w, h in sizes]
    got = ctx.render_batch(which, poses, ks, [w for w, _ in sizes], [h for _, h in sizes], fmt="f32", tile=(16, 16),
                           batch_depth=64)
    for s, p, k, (w, h), img in zip(which, poses, ks, sizes, got):
        np.testing.assert_array_equal(img, ctx.render(s, p, k, w, h, fmt="f32", tile=(16, 16)))
    assert not got[2].any()
    for s in scenes:
        s.free()


@pytest.mark.parametrize("n,views", [(180_000, 46), (180_000, 48)])
def test_depth_buckets_of_more_segments_than_a_round(ctx, n, views):
    """About 506 segments, each forming the samples' distribution, and 528,
    which read it: every view is its single frame."""
    rng = np.random.default_rng(5)
    z = rng.uniform(2.0, 30.0, n)
    xy = rng.uniform(-0.7, 0.7, (n, 2))
    scene = make_scene(np.column_stack([xy[:, 0] * z, xy[:, 1] * z, z]),
                       np.repeat(np.log(0.01 * z)[:, None], 3, axis=1), None, rng.normal(-1.0, 1.0, n),
                       rng.uniform(0.0, 1.0, (n, 3)))
    s = ctx.load_scene(scene)
    poses = [synth.Pose(np.eye(3, dtype=np.float32), np.array([0.01 * i, 0, -0.2 * i], np.float32))
             for i in range(views)]
    k, W, H = intr(40.0, 33, 30), 66, 60
    _say("many segments", n, views)
    got = ctx.render_batch([s] * views, poses, [k] * views, [W] * views, [H] * views, fmt="f32", tile=(16, 16))
    for i in (0, 1, views // 2, views - 1):
        want = ctx.render(s, poses[i], k, W, H, fmt="f32", tile=(16, 16))
        assert want.any()
        np.testing.assert_array_equal(got[i], want)
    s.free()


def _rect_scene(kind, n):
    """Gaussians whose tile rectangles meet the placement in different forms."""
    rng = np.random.default_rng(n + 1)
    z = rng.uniform(2.0, 6.0, n)
    size = {"small": 0.004, "wide": 0.25}.get(kind, 0.02)
    ls = np.repeat(np.log(size * z)[:, None], 3, axis=1) + rng.normal(0.0, 0.3, (n, 3))
    if kind == "mixed":  # a few, near ones among them, over the whole frame
        ls[:: max(1, n // 9)] = 1.0
    xy = rng.uniform(-1.0, 1.0, (n, 2)) * np.array([1.0, 0.6])
    if kind == "stack":  # all on a few tiles
        xy = rng.normal(0.0, 0.01, (n, 2))
    means = np.column_stack([xy[:, 0] * z, xy[:, 1] * z, z])
    return make_scene(means, ls, None, rng.normal(0.0, 1.0, n), rng.uniform(0.0, 1.0, (n, 3)))


@pytest.mark.parametrize("kind", ["small", "wide", "mixed", "stack"])
@pytest.mark.parametrize("size,tile", [((40, 24), (16, 16)), ((500, 300), (8, 8)), ((1000, 900), (8, 8)),
                                       ((2048, 40), (8, 8)), ((24, 2048), (8, 8)), ((1100, 700), (16, 32))])
def test_tile_placement_of_every_grid_form(ctx, size, tile, kind):
    """Grids of one group of tile rows and of several, of one row or column,
    of 256 tiles across; rectangles of one tile, of many, and of the whole
    frame; lists and ranges of the plain 64-bit key sort."""
    W, H = size
    n = 700 if kind in ("wide", "mixed") else 6000
    scene = _rect_scene(kind, n)
    s = ctx.load_scene(scene)
    _say("tile placement", size, tile, kind)
    dbg = ctx.render_debug(s, eye_pose(), intr(max(W, H) / 2.0, W / 2, H / 2), W, H, tile=tile)
    assert dbg["n_dup"] > 0
    gc.check_tiles(dbg, *tile)
    s.free()


def test_tile_placement_of_uneven_views_in_one_batch(ctx):
    """Views of different grids (one, and several groups of tile rows), loads
    and scenes, one without a Gaussian: each frame is the view's own, with the
    counting placement and with the radix passes."""
    a, b = ctx.load_scene(_rect_scene("mixed", 700)), ctx.load_scene(_rect_scene("small", 6000))
    which, sizes = [a, b, b, a, b], [(1000, 900), (40, 24), (33, 500), (300, 200), (64, 64)]
    poses = [eye_pose()] * 4 + [synth.Pose(np.eye(3, dtype=np.float32), np.array([0, 0, 50.0], np.float32))]
    ks = [intr(max(w, h) / 2.0, w / 2, h / 2) for w, h in sizes]
    for tile in ((8, 8), (16, 32)):
        got = {}
        for binning in (True, False):
            ctx.set_tile_binning(binning)
            try:
                got[binning] = ctx.render_batch(which, poses, ks, [w for w, _ in sizes], [h for _, h in sizes],
                                                fmt="f32", tile=tile, batch_depth=64)
            finally:
                ctx.set_tile_binning(True)
        for i, (w, h) in enumerate(sizes):
            want = ctx.render(which[i], poses[i], ks[i], w, h, fmt="f32", tile=tile)
            np.testing.assert_array_equal(got[True][i], want)
            np.testing.assert_array_equal(got[False][i], want)
        assert not got[True][4].any()
    a.free()
    b.free()


@pytest.mark.parametrize("kind", ["small", "mixed"])
@pytest.mark.parametrize("size,tile", [((512, 512), (16, 16)), ((513, 512), (16, 16)), ((1030, 1030), (16, 16)),
                                       ((2100, 1300), (8, 8)), ((4096, 24), (8, 8)), ((4104, 24), (8, 8)),
                                       ((1933, 1083), (16, 32)), ((1083, 1933), (32, 16))])
def test_tiles_sharing_a_list_give_the_same_frame(ctx, size, tile, kind):
    """At the limit of one tile per list and beyond, with lists that hang over
    the frame's edges, the most tiles per list, and a grid too wide for the
    counting placement even so: the frame of the radix passes, whose tiles
    have lists of their own."""
    W, H = size
    s = ctx.load_scene(_rect_scene(kind, 6000 if kind == "small" else 700))
    k = intr(max(W, H) / 2.0, W / 2, H / 2)
    _say("shared lists", size, tile, kind)
    got, st = {}, {}
    for binning in (True, False):
        ctx.set_tile_binning(binning)
        try:
            got[binning] = ctx.render(s, eye_pose(), k, W, H, fmt="f32", tile=tile)
            st[binning] = ctx.stats()
        finally:
            ctx.set_tile_binning(True)
    np.testing.assert_array_equal(got[True], got[False])
    assert got[True].any()
    for name in ("duplicates", "tiles", "visible"):
        assert st[True][name] == st[False][name]
    s.free()


@pytest.mark.parametrize("size,tile", [((1030, 1030), (16, 16)), ((1933, 1083), (16, 32))])
def test_shared_lists_with_four_depth_passes(ctx, size, tile):
    """Tiles that share lists, in the depth order of the radix passes: the
    frame and the counts, those of the allocation-free form too, are those of
    the bucketed order."""
    import torch
    W, H = size
    s = ctx.load_scene(_rect_scene("small", 6000))
    k = intr(max(W, H) / 2.0, W / 2, H / 2)
    _say("shared lists, four passes", size, tile)
    got, st, cnt = {}, {}, {}
    for passes in (3, 4):
        ctx.set_depth_passes(passes)
        try:
            got[passes] = ctx.render(s, eye_pose(), k, W, H, fmt="f32", tile=tile)
            st[passes] = ctx.stats()
            out = torch.empty((H, W, 3), dtype=torch.float32, device="cuda")
            counters = torch.zeros(6, dtype=torch.int32, device="cuda")
            ctx.render_noalloc(s, eye_pose(), k, W, H, out, counters=counters, fmt="f32", tile=tile)
            torch.cuda.synchronize()
            cnt[passes] = counters.cpu().numpy()[:4].tolist()
        finally:
            ctx.set_depth_passes(3)
        np.testing.assert_array_equal(out.cpu().numpy(), got[3])
    np.testing.assert_array_equal(got[3], got[4])
    assert (st[3]["sort_passes"], st[4]["sort_passes"]) == (4, 5)
    for name in ("duplicates", "tiles", "visible", "fallbacks"):
        assert st[3][name] == st[4][name]
    assert cnt[3] == cnt[4] == [st[3]["duplicates"], st[3]["visible"], st[3]["fallbacks"], 0]
    s.free()


@pytest.mark.parametrize("how", ["culled", "radix", "counted"])
def test_scratch_of_the_placement_is_kept_only_where_it_is_used(how):
    """A large frame of small tiles: its buffers take what its records, its 2^20
    entries (six words each) and its tiles need, not a row of all tiles per unit
    (1 MB a row for 512 x 512 tiles) where the lists are not placed by counting,
    nor beside the keys where they are."""
    import torch
    W = H = 4096
    out = torch.zeros((H, W, 3), dtype=torch.uint8, device="cuda")
    c = tigas.Context(0)
    try:
        s = c.load_scene(_rect_scene("small", 6000))
        c.set_tile_culling(how == "culled")
        c.set_tile_binning(how != "radix")
        tile = (16, 32) if how == "counted" else (8, 8)
        k = intr(W / 2.0, W / 2, H / 2)
        c.render(s, eye_pose(), intr(20.0, 16, 16), 32, 32, tile=(8, 8))  # the kernels are loaded
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        c.render(s, eye_pose(), k, W, H, out=out, tile=tile)
        torch.cuda.synchronize()
        used = before - torch.cuda.mem_get_info()[0]
        _say("placement scratch", how, used >> 20, "MiB")
        assert out.any() and used < 64 << 20
    finally:
        c.close()


@pytest.mark.parametrize("kind", ["small", "mixed", "stack"])
@pytest.mark.parametrize("size", [(320, 320), (317, 331), (448, 448), (451, 449)])
def test_blend_by_quarters_halves_and_whole_blocks(ctx, size, kind):
    """One, two and three views of one frame in a launch: few blocks are
    composited by quarters, some by halves, many whole, with blocks that hang
    over the frame's edges; the frame is the same."""
    W, H = size
    s = ctx.load_scene(_rect_scene(kind, 6000 if kind != "mixed" else 700))
    k = intr(max(W, H) / 2.0, W / 2, H / 2)
    _say("blend parts", size, kind)
    want = ctx.render(s, eye_pose(), k, W, H, fmt="f32", bg=(0.1, 0.6, 0.3), tile=(16, 16))
    for n in (2, 3):
        for got in ctx.render_batch([s] * n, [eye_pose()] * n, [k] * n, [W] * n, [H] * n, fmt="f32",
                                    bg=(0.1, 0.6, 0.3), tile=(16, 16)):
            np.testing.assert_array_equal(got, want)
    small = ctx.render(s, eye_pose(), intr(40.0, 33, 30), 66, 60, fmt="f32", bg=(0.1, 0.6, 0.3), tile=(16, 16))
    n = 60  # 4320 blocks in all
    for got in ctx.render_batch([s] * n, [eye_pose()] * n, [intr(40.0, 33, 30)] * n, [66] * n, [60] * n, fmt="f32",
                                bg=(0.1, 0.6, 0.3), tile=(16, 16)):
        np.testing.assert_array_equal(got, small)
    s.free()


@pytest.mark.parametrize("opacity", [0.02, 0.6, 0.9999])
@pytest.mark.parametrize("n", [1, 7, 8, 9, 63, 64, 65, 71, 72, 73, 129, 700])
def test_blend_groups_and_batches(ctx, n, opacity):
    """Lists around the sizes of a group and of a batch, of Gaussians over the
    whole frame (wide ones, whose exponents span little, among narrow ones),
    that stop no pixel, stop pixels inside groups, and reach the cap on alpha:
    the oracle's frame, and the same one from every tile shape, with and
    without the lists' cells."""
    rng = np.random.default_rng(n)
    W, H = 50, 41
    z = rng.uniform(2.0, 6.0, n)
    xy = rng.uniform(-1.0, 1.0, (n, 2)) * np.array([1.0, 0.8])
    ls = np.repeat(np.log(rng.choice([0.03, 0.3, 2.0], n) * z)[:, None], 3, axis=1) + rng.normal(0.0, 0.2, (n, 3))
    scene = make_scene(np.column_stack([xy[:, 0] * z, xy[:, 1] * z, z]), ls, None,
                       np.full(n, math.log(opacity / (1.0 - opacity))), rng.uniform(0.0, 1.0, (n, 3)))
    s = ctx.load_scene(scene)
    k = intr(W / 2.0, W / 2, H / 2)
    bg = (0.2, 0.5, 0.9)
    _say("blend groups", n, opacity)
    img = ctx.render(s, eye_pose(), k, W, H, fmt="f32", bg=bg, tile=(16, 16))
    br, nb = orc.render_frame(orc.preprocess(scene, eye_pose(), k, W, H), bg=bg)
    res = gc.check_frame_pixels(img.reshape(-1, 3), br.reshape(-1, br.shape[2], 4), nb.reshape(-1))
    # (pixels with more decision forks than the oracle follows cannot be judged)
    assert res["n_bad"] <= res["n_unresolved"] <= W * H // 50, res
    for tile in ((8, 8), (16, 32), (32, 16)):
        np.testing.assert_array_equal(ctx.render(s, eye_pose(), k, W, H, fmt="f32", bg=bg, tile=tile), img)
    ctx.set_tile_binning(False)
    try:
        np.testing.assert_array_equal(ctx.render(s, eye_pose(), k, W, H, fmt="f32", bg=bg, tile=(16, 16)), img)
    finally:
        ctx.set_tile_binning(True)
    s.free()


@pytest.mark.parametrize("tile", [(16, 16), (8, 8), (16, 32), (32, 16)])
def test_culled_tile_lists_bit_exact_and_frames_unchanged(ctx, c1, tile):
    """Tighter tile culling: the lists equal the reference less exactly the
    entries its tile test drops, fewer entries are sorted, and the frame is
    bit-identical to the one rendered from whole rectangles."""
    scene, poses, k, W, H = c1
    s = ctx.load_scene(scene)
    ctx.set_tile_culling(True)
    try:
        dbg = ctx.render_debug(s, poses[0], k, W, H, tile=tile)
        culled = ctx.render(s, poses[0], k, W, H, fmt="f32", tile=tile)
        d_culled = ctx.stats()["duplicates"]
    finally:
        ctx.set_tile_culling(False)
    gc.check_tiles(dbg, *tile, cull=True)
    full = ctx.render(s, poses[0], k, W, H, fmt="f32", tile=tile)
    d_full = ctx.stats()["duplicates"]
    _say("culled", tile, d_culled, "of", d_full)
    np.testing.assert_array_equal(culled, full)
    assert d_culled == dbg["n_dup"] and d_culled < d_full


def test_c1_frame_matches_oracle(ctx, c1):
    scene, poses, k, W, H = c1
    s = ctx.load_scene(scene)
    img = ctx.render(s, poses[0], k, W, H, fmt="f32")
    proj = orc.preprocess(scene, poses[0], k, W, H)
    br, nb = orc.render_frame(proj)
    res = gc.check_frame_pixels(img.reshape(-1, 3), br.reshape(-1, br.shape[2], 4), nb.reshape(-1))
    _say("c1 frame", res)
    assert res["n_bad"] == 0 and res["n_unresolved"] == 0, res
    st = ctx.stats()
    _say("stats", st)
    assert st["visible"] > 0 and st["duplicates"] > 0


def test_c1_rgb8_is_the_packed_f32_frame(ctx, c1):
    scene, poses, k, W, H = c1
    s = ctx.load_scene(scene)
    f = ctx.render(s, poses[0], k, W, H, fmt="f32", bg=(0.2, 0.3, 0.4))
    b = ctx.render(s, poses[0], k, W, H, fmt="rgb8", bg=(0.2, 0.3, 0.4))
    # the 8-bit frame is the oracle's pack of the FP32 frame, bit for bit ...
    np.testing.assert_array_equal(b, orc.pack_rgb8(f))
    # ... and within one level of the pack of the FP64 oracle's own frame
    proj = orc.preprocess(scene, poses[0], k, W, H)
    nominal = orc.render_nominal(proj, bg=(0.2, 0.3, 0.4)).astype(np.float32)
    assert np.abs(b.astype(int) - orc.pack_rgb8(nominal).astype(int)).max() <= 1


def test_frames_bit_identical_across_tiles_and_batch_depths(ctx, c1):
    scene, poses, k, W, H = c1
    s = ctx.load_scene(scene)
    ref = ctx.render(s, poses[0], k, W, H, fmt="f32")
    for tile in [(8, 8), (16, 16), (16, 32), (32, 16)]:
        for bd in (64, 128, 256):
            for ppl in ((1,) if tile[1] < 16 else (1, 2)):
                got = ctx.render(s, poses[0], k, W, H, fmt="f32", tile=tile, batch_depth=bd, ppl=ppl)
                np.testing.assert_array_equal(got, ref, err_msg=f"tile={tile} bd={bd} ppl={ppl}")


def test_render_is_deterministic(ctx, c1):
    scene, poses, k, W, H = c1
    s = ctx.load_scene(scene)
    a = ctx.render(s, poses[0], k, W, H, fmt="f32")
    b = ctx.render(s, poses[0], k, W, H, fmt="f32")
    np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("size", [(1, 1), (7, 13), (33, 17), (100, 1)])
def test_ragged_and_tiny_images(ctx, size):
    W, H = size
    rng = np.random.default_rng(W * 100 + H)
    scene = random_tiny_scene(rng, n=300, extent=1.0)
    k = intr(max(W, H) * 0.9, W / 2, H / 2)
    s = ctx.load_scene(scene)
    _say("ragged", size)
    for tile in [(16, 16), (8, 8)]:
        dbg = ctx.render_debug(s, eye_pose(), k, W, H, tile=tile)
        gc.check_tiles(dbg, *tile)
        proj = orc.preprocess(scene, eye_pose(), k, W, H)
        gc.check_preprocess(dbg, proj, W, H)
        br, nb = orc.render_frame(proj)
        res = gc.check_frame_pixels(dbg["image"].reshape(-1, 3), br.reshape(-1, br.shape[2], 4), nb.reshape(-1))
        assert res["n_bad"] == 0 and res["n_unresolved"] == 0, res


@pytest.mark.parametrize("size", [(2048, 24), (2072, 24), (24, 2072)])
def test_wide_views_both_rectangle_encodings(ctx, size):
    # up to 256 x 256 tiles a view's tile rectangles travel packed in one word
    # through the depth passes; beyond that (here 259 tiles of 8 px) the last
    # depth pass gathers them: lists and pixels must match either way
    W, H = size
    rng = np.random.default_rng(W + 7 * H)
    scene = random_tiny_scene(rng, n=400, extent=1.0)
    axis = 0 if W > H else 1
    scene.means[:, axis] *= 7.0
    k = intr(700.0, W / 2, H / 2)
    s = ctx.load_scene(scene)
    _say("wide", size)
    dbg = ctx.render_debug(s, eye_pose(), k, W, H, tile=(8, 8))
    gc.check_tiles(dbg, 8, 8)
    proj = orc.preprocess(scene, eye_pose(), k, W, H)
    gc.check_preprocess(dbg, proj, W, H)
    br, nb = orc.render_frame(proj)
    res = gc.check_frame_pixels(dbg["image"].reshape(-1, 3), br.reshape(-1, br.shape[2], 4), nb.reshape(-1))
    assert res["n_bad"] == 0 and res["n_unresolved"] == 0, res
    assert dbg["n_dup"] > 0
    if max(W, H) > 2048:  # Gaussians reach the tiles past 255
        assert dbg["bbox"][:, 2 + axis].max() >= 2048


def test_empty_scene_and_all_culled_render_background(ctx):
    bg = (0.25, 0.5, 0.75)
    empty = make_scene(np.zeros((0, 3)))
    s = ctx.load_scene(empty)
    img = ctx.render(s, eye_pose(), intr(50, 20, 20), 40, 40, fmt="f32", bg=bg)
    np.testing.assert_array_equal(img, np.broadcast_to(np.float32(bg), img.shape))
    behind = make_scene([[0, 0, -3], [0, 0, 0.1], [50, 0, 3]], log_scales=[[math.log(0.3)] * 3] * 3)
    s2 = ctx.load_scene(behind)
    img = ctx.render(s2, eye_pose(), intr(50, 20, 20), 40, 40, fmt="f32", bg=bg)
    np.testing.assert_array_equal(img, np.broadcast_to(np.float32(bg), img.shape))
    assert ctx.stats()["duplicates"] == 0


def test_nan_and_zero_quaternion_are_dropped(ctx):
    sc = make_scene([[0, 0, 3], [0.1, 0, 3], [0, 0.1, 3], [0, 0, 4], [0.05, 0.05, 3], [-0.1, 0, 3.5],
                     [0, -0.1, 3.5]], log_scales=[[math.log(0.2)] * 3] * 7,
                    logits=[2] * 7, colors=[[1, 0, 0], [0, 1, 0], [0, 0, 1], [1, 1, 1]] + [[0.5, 0.5, 0.5]] * 3,
                    sh_degree=3)
    sc.quats[1] = 0
    sc.means[2, 1] = np.nan
    sc.log_scales[3, 0] = np.inf
    sc.sh[4, 12, 1] = np.nan          # a degree-3 coefficient
    sc.sh[5, 0, 2] = -np.inf          # the DC term
    sc.opacity_logits[6] = np.inf
    s = ctx.load_scene(sc)
    k = intr(60, 16, 16)
    img = ctx.render(s, eye_pose(), k, 32, 32, fmt="f32")
    proj = orc.preprocess(sc, eye_pose(), k, 32, 32)
    np.testing.assert_array_equal(proj.valid, [True, False, False, False, False, False, False])
    assert np.isfinite(img).all()
    br, nb = orc.render_frame(proj)
    res = gc.check_frame_pixels(img.reshape(-1, 3), br.reshape(-1, br.shape[2], 4), nb.reshape(-1))
    assert res["n_bad"] == 0 and res["n_unresolved"] == 0, res


def test_closed_form_saturated_layers(ctx):
    bg = (0.1, 0.2, 0.3)
    c1c = np.array([0.9, 0.8, 0.7])
    sc = make_scene([[0, 0, 2], [0, 0, 3], [0, 0, 4]], log_scales=[[math.log(5.0)] * 3] * 3,
                    logits=[10.0] * 3, colors=[c1c, [0, 1, 0], [1, 0, 0]])
    s = ctx.load_scene(sc)
    img = ctx.render(s, eye_pose(), intr(50, 4, 4), 8, 8, fmt="f32", bg=bg).astype(np.float64)
    col = 0.5 + (0.5 / math.sqrt(math.pi)) * sc.sh[0, 0].astype(np.float64)
    want = float(np.float32(0.99)) * col + (1 - float(np.float32(0.99))) * np.array(bg)
    np.testing.assert_allclose(img, np.broadcast_to(want, img.shape), atol=1e-6)


def test_rungs_and_principal_point(ctx, c1):
    scene, poses, k, W, H = c1
    s = ctx.load_scene(scene)
    for sc in (0.25, 0.5, 0.75):
        img = ctx.render(s, poses[0], k, W, H, res_scale=sc, fmt="f32")
        proj = orc.preprocess(scene, poses[0], k, W, H, scale=sc)
        assert img.shape[:2] == (proj.out_h, proj.out_w)
        br, nb = orc.render_frame(proj)
        res = gc.check_frame_pixels(img.reshape(-1, 3), br.reshape(-1, br.shape[2], 4), nb.reshape(-1))
        _say("rung", sc, res)
        assert res["n_bad"] == 0 and res["n_unresolved"] == 0, res


def test_invalid_arguments_are_reported(ctx, c1):
    scene, poses, k, W, H = c1
    s = ctx.load_scene(scene)
    with pytest.raises(tigas.TigasError, match="E_INVALID"):
        ctx.render(s, poses[0], k, W, H, tile=(12, 12))
    with pytest.raises(tigas.TigasError, match="E_INVALID"):
        ctx.render(s, poses[0], k, 0, H)
    bad = synth.Pose(np.full((3, 3), np.nan, np.float32), np.zeros(3, np.float32))
    with pytest.raises(tigas.TigasError, match="E_INVALID"):
        ctx.render(s, bad, k, W, H)
    # an SH degree above the scene's is refused, not clamped
    with pytest.raises(tigas.TigasError, match="E_INVALID"):
        ctx.render(s, poses[0], k, W, H, sh_degree=4)
    s1 = ctx.load_scene(dataclasses.replace(scene, sh_degree=1))
    with pytest.raises(tigas.TigasError, match="E_INVALID"):
        ctx.render(s1, poses[0], k, W, H, sh_degree=2)
    s1.free()


@pytest.mark.parametrize("fmt,scale", [("rgb8", 1.0), ("f32", 0.5)])
def test_small_output_buffer_reports_the_frame_size(ctx, c1, fmt, scale):
    # E_BUFFER for a frame buffer below out_w * out_h * 3 * (1 or 4) bytes;
    # out_w and out_h are written all the same
    scene, poses, k, W, H = c1
    s = ctx.load_scene(scene)
    ow, oh = tigas.output_size(W, H, scale)
    need = ow * oh * 3 * (4 if fmt == "f32" else 1)
    buf = np.zeros(need - 1, np.uint8)
    q = tigas.quality_c(scale, -1, fmt)
    fr = tigas.FrameC(ctypes.c_void_p(buf.ctypes.data), buf.nbytes, 0, 0, 0)
    L = tigas.lib()
    rc = L.tigas_render(s.handle, ctypes.byref(tigas.pose_c(poses[0])), ctypes.byref(tigas.intr_c(k)), W, H,
                        ctypes.byref(q), ctypes.byref(fr), None)
    assert rc == -4, rc
    assert (fr.out_w, fr.out_h) == (ow, oh)
    assert "too small" in L.tigas_last_error().decode()
    assert not buf.any()        # nothing was written
    s.free()


@pytest.mark.parametrize("deg", [0, 1, 2])
def test_scenes_of_lower_sh_degree_match_oracle(ctx, c1, deg):
    # a degree-d scene stores only its (d+1)^2 coefficients
    scene, poses, k, W, H = c1
    sc = dataclasses.replace(scene, sh_degree=deg)
    s = ctx.load_scene(sc)
    img = ctx.render(s, poses[0], k, W, H, fmt="f32")
    proj = orc.preprocess(sc, poses[0], k, W, H)
    br, nb = orc.render_frame(proj)
    res = gc.check_frame_pixels(img.reshape(-1, 3), br.reshape(-1, br.shape[2], 4), nb.reshape(-1))
    _say("scene degree", deg, res)
    assert res["n_bad"] == 0 and res["n_unresolved"] == 0, res
    s.free()


@pytest.mark.parametrize("req", [0, 1, 2, 3])
def test_request_sh_degree_at_or_below_the_scenes_matches_oracle(ctx, c1, req):
    scene, poses, k, W, H = c1
    s = ctx.load_scene(scene)
    img = ctx.render(s, poses[0], k, W, H, fmt="f32", sh_degree=req)
    proj = orc.preprocess(scene, poses[0], k, W, H, sh_degree=req)
    br, nb = orc.render_frame(proj)
    res = gc.check_frame_pixels(img.reshape(-1, 3), br.reshape(-1, br.shape[2], 4), nb.reshape(-1))
    _say("request degree", req, res)
    assert res["n_bad"] == 0 and res["n_unresolved"] == 0, res
    s.free()


def _needle_scene(n=40, seed=41):
    """Long thin splats lying in planes facing the camera, their long axis at
    angles across the image plane: seen that way their 2D covariance is close
    to singular (a*c/det far above 64) unless the axis is nearly horizontal or
    vertical."""
    rng = np.random.default_rng(seed)
    means = np.column_stack([rng.uniform(-0.5, 0.5, n), rng.uniform(-0.5, 0.5, n), rng.uniform(2.5, 4.0, n)])
    ls = np.column_stack([np.log(rng.uniform(0.08, 0.4, n)), np.log(rng.uniform(1e-4, 3e-3, n)),
                          np.log(rng.uniform(1e-4, 3e-3, n))])
    ang = rng.uniform(0.0, math.pi, n)
    tilt = rng.normal(0.0, 0.05, (n, 2))
    q = np.column_stack([np.cos(ang / 2), tilt[:, 0], tilt[:, 1], np.sin(ang / 2)])
    cols = rng.uniform(0.0, 1.0, (n, 3))
    return make_scene(means, ls, q, rng.normal(1.0, 1.0, n), cols, sh_degree=0)


def test_fp64_fallback_conics_and_pixels_match_oracle(ctx):
    sc = _needle_scene()
    k = intr(220.0, 64, 64)
    s = ctx.load_scene(sc)
    dbg = ctx.render_debug(s, eye_pose(), k, 128, 128)
    st = ctx.stats()
    proj = orc.preprocess(sc, eye_pose(), k, 128, 128)
    sure_fb, _ = gc.fallback_sets(proj)
    vis = dbg["touched"] > 0
    err = gc.check_preprocess(dbg, proj, 128, 128)      # fallback conics within 1e-6 relative
    _say("fallbacks", st["fallbacks"], "sure", int(sure_fb.sum()), err)
    assert int(np.sum(sure_fb & vis)) >= 10
    assert st["fallbacks"] >= int(np.sum(sure_fb & vis))
    br, nb = orc.render_frame(proj)
    res = gc.check_frame_pixels(dbg["image"].reshape(-1, 3), br.reshape(-1, br.shape[2], 4), nb.reshape(-1))
    _say("needles frame", res)
    assert res["n_bad"] == 0 and res["n_unresolved"] == 0, res
    s.free()


def test_kernel_timing_brackets_every_launch(ctx, c1):
    scene, poses, k, W, H = c1
    s = ctx.load_scene(scene)
    ref = ctx.render(s, poses[0], k, W, H, fmt="f32")
    ctx.profile_kernels(True)
    try:
        for _ in range(3):
            got = ctx.render(s, poses[0], k, W, H, fmt="f32")
        kt = ctx.kernel_times()
    finally:
        ctx.profile_kernels(False)
    _say("kernel times", kt)
    np.testing.assert_array_equal(got, ref)
    pre = [n for n in kt if "k_preprocess<0, 3>" in n]
    blend = [n for n in kt if "k_blend<" in n]
    assert len(pre) == 1 and kt[pre[0]][0] == 3
    assert len(blend) == 1 and kt[blend[0]][0] == 3
    assert all(ms > 0 for _, ms in kt.values())


def test_block_culling_never_changes_a_pixel(ctx, monkeypatch):
    # the blend drops, per wave, entries whose exponent stays below the skip
    # threshold on its whole block; frames must equal those rendered without it
    scene = synth.c3_scene()
    traj = synth.c3_trajectory(300)
    k = synth.fov_intrinsics(1920, 1080)
    monkeypatch.setenv("TIGAS_BLEND_CULL", "0")
    plain = tigas.Context(0)
    monkeypatch.delenv("TIGAS_BLEND_CULL")
    try:
        sa = ctx.load_scene(scene)
        sb = plain.load_scene(scene)
        for i in (0, 75, 150, 225):
            for tile, ppl in (((16, 32), 1), ((16, 16), 2), ((8, 8), 1)):
                _say("cull check pose", i, tile, ppl)
                a = ctx.render(sa, traj[i], k, 1920, 1080, fmt="f32", tile=tile, batch_depth=64, ppl=ppl)
                b = plain.render(sb, traj[i], k, 1920, 1080, fmt="f32", tile=tile, batch_depth=64, ppl=ppl)
                np.testing.assert_array_equal(a, b, err_msg=f"pose {i} tile {tile} ppl {ppl}")
        ea, ca = ctx.count_blend_work(sa, traj[0], k, 1920, 1080, tile=(16, 32), batch_depth=64, ppl=1)
        eb, cb = plain.count_blend_work(sb, traj[0], k, 1920, 1080, tile=(16, 32), batch_depth=64, ppl=1)
        _say("evaluations with / without culling", ea, eb, "contributions", ca, cb)
        assert ca == cb and ea <= eb
        sa.free()
        sb.free()
    finally:
        plain.close()
