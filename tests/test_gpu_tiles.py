"""Tile sizes other than 16x16 (one key bin per tw x th tile, one wave per 16x16 sub-tile) and
the native tile autotuner, against the CPU oracle run at the same tile size.

Keys, values, ranges and n_contrib depend on the tile size and must match the oracle's
bit-exactly; images within 1e-4 of the oracle at the same tile size, gradients within the
per-tensor bound of the 16x16 tests.  (Images themselves depend slightly on the tile size: a
Gaussian reaches a pixel only if its 3-sigma rectangle, rounded out to whole tiles, covers the
pixel's tile, and its alpha can stay above 1/255 a little beyond 3 sigma.)
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import IMG_TOL, assert_grad_close, excluded_pixels, log, make_ctx, to_gpu
from test_gpu_parity import BG, large_footprint_sub, small_multiview

pytestmark = pytest.mark.gpu

TILES = [(32, 16), (16, 32), (32, 32), (64, 32), (64, 64), (16, 16, 8), (32, 32, 8)]
CASES = {
    "multiview_sh3_ragged": lambda: small_multiview(),
    "tiny_dense": lambda: synth.tiny_scene(2, 300, 40, 36, sh_degree=2, log_scale_mu=-2.0),
    "large_footprint_64_4x32x32": large_footprint_sub,
}


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("case", list(CASES))
def test_tile_keys_images_match_oracle(case, tile):
    scene, cams, _ = CASES[case]()
    log(f"[tile {tile}] {case}")
    g = to_gpu(scene)
    ctx = make_ctx(scene.n, cams)
    ctx.tile = tile
    out = ctx.render_fwd(g, cams, BG)
    ctx.sync()
    tile = tile[:2]  # the sub-tile split is internal to the blend; the definition has the tile size
    for v, cam in enumerate(cams):
        p = oracle.project(scene, cam, tile)
        assert not np.any(p.flags & oracle.FLAG_RADIUS)
        k, val, r = oracle.keys(p, cam, tile)
        TX, TY = oracle.tiles_of(cam, tile)
        gk, gv, gr = ctx.debug_keys(v, k.size + 16, TX * TY)
        np.testing.assert_array_equal(gk, k)
        np.testing.assert_array_equal(gv, val)
        np.testing.assert_array_equal(gr, r)
        vr = oracle.render_view(scene, cam, bg=BG, tile=tile, proj=p, key_data=(k, val, r))
        ex = excluded_pixels(vr, cam, tile=tile)
        assert np.abs(out[v].rgb.cpu().numpy() - vr.rgb)[:, ~ex].max() <= IMG_TOL
        assert np.abs(out[v].t_final.cpu().numpy() - vr.t_final)[~ex].max() <= IMG_TOL
        np.testing.assert_array_equal(out[v].n_contrib.cpu().numpy()[~ex], vr.n_contrib[~ex])
        assert ex.mean() <= 0.01


@pytest.mark.parametrize("tile", [(32, 32), (64, 32), (16, 16, 8)])
@pytest.mark.parametrize("case", ["multiview_sh3_ragged", "large_footprint_64_4x32x32"])
def test_tile_gradients_match_oracle(case, tile):
    scene, cams, dls = CASES[case]()
    log(f"[tile grad {tile}] {case}")
    gtile, tile = tile, tile[:2]
    renders = [oracle.render_view(scene, c, bg=BG, tile=tile) for c in cams]
    dls = [d.copy() for d in dls]
    for d, vr, cam in zip(dls, renders, cams):
        d[:, excluded_pixels(vr, cam, grad=True, tile=tile)] = 0.0
    og, _, ogn, ocnt = oracle.render_backward(scene, cams, dls, bg=BG, tile=tile, renders=renders)
    g = to_gpu(scene)
    ctx = make_ctx(scene.n, cams)
    ctx.tile = gtile
    out = ctx.render_fwd(g, cams, BG)
    grads = g.zeros_like()
    gn = torch.zeros(g.capacity, device="cuda")
    cnt = torch.zeros(g.capacity, dtype=torch.int32, device="cuda")
    ctx.render_bwd(g, cams, BG, out, [torch.as_tensor(d, device="cuda") for d in dls], grads, gn, cnt)
    ctx.sync()
    gflag = np.zeros(scene.n, bool)
    for cam in cams:
        gflag |= (oracle.project(scene, cam, tile).flags & oracle.GAUSS_GRAD_FLAGS) != 0
    for name in ("mean", "quat", "log_scale", "logit", "sh"):
        got = getattr(grads, name)[..., :scene.n].cpu().numpy()
        rel = assert_grad_close(name, got, getattr(og, name), exclude=gflag)
        log(f"  {name}: max rel err (significant) {rel:.2e}")
    np.testing.assert_array_equal(cnt[:scene.n].cpu().numpy(), ocnt)
    assert_grad_close("gradnorm", gn[:scene.n].cpu().numpy(), ogn, exclude=gflag)


@pytest.mark.parametrize("tile", [(16, 16), (32, 32)])
def test_subtile8_forward_matches_subtile16(tile):
    """8x8 sub-tiles (one pixel per lane) walk the same lists in the same order as 16x16
    sub-tiles; only the float32 rounding of the pixel offsets differs (they are formed relative
    to the sub-tile's origin), so images agree to float32 rounding and n_contrib everywhere but
    at decisions within rounding of a threshold."""
    scene, cams, dls = small_multiview(seed=9, n=2500, views=2, W=150, H=110)
    g = to_gpu(scene)
    outs = []
    for sub in (16, 8):
        ctx = make_ctx(scene.n, cams)
        ctx.tile = (*tile, sub)
        outs.append(ctx.render_fwd(g, cams, BG))
        ctx.sync()
    for a, b in zip(*outs):
        assert (a.rgb - b.rgb).abs().max().item() <= 1e-5
        assert (a.t_final - b.t_final).abs().max().item() <= 1e-5
        assert (a.n_contrib != b.n_contrib).float().mean().item() <= 1e-3


def test_backward_rejects_a_tile_size_other_than_the_forwards():
    from paper_2411_14847_amd import DassError
    scene, cams, dls = small_multiview(seed=4, n=500, views=2, W=64, H=48)
    g = to_gpu(scene)
    ctx = make_ctx(scene.n, cams)
    ctx.tile = (32, 32)
    out = ctx.render_fwd(g, cams, BG)
    ctx.tile = (16, 16)
    with pytest.raises(DassError):
        ctx.render_bwd(g, cams, BG, out, [torch.as_tensor(d, device="cuda") for d in dls], g.zeros_like())
    ctx.tile = (48, 16)
    with pytest.raises(DassError):
        ctx.render_fwd(g, cams, BG)
    ctx.sync()


def test_autotuner_picks_a_timed_candidate_and_keeps_parity():
    scene, cams, dls = small_multiview(seed=6, n=4000, views=3, W=320, H=200)
    g = to_gpu(scene)
    ctx = make_ctx(scene.n, cams)
    out = ctx.render_fwd(g, cams, BG)
    dl_t = [torch.as_tensor(d, device="cuda") for d in dls]
    scratch = g.zeros_like()
    res = ctx.autotune_tile(g, cams, BG, out, dl_t, scratch, reps=2)
    log(f"  autotune: {res}; chose {ctx.tile}")
    assert ctx.tile in res and res[ctx.tile] is not None
    fastest = min(v for v in res.values() if v is not None)
    # the library's rule, in its float32 arithmetic: the first candidate within 1% of the fastest
    lim = np.float32(1.01) * np.float32(fastest)
    first_close = next(c for c, v in res.items() if v is not None and np.float32(v) <= lim)
    assert ctx.tile == first_close
    out = ctx.render_fwd(g, cams, BG)
    ctx.sync()
    tile = ctx.tile[:2]  # a third entry is the blend's sub-tile size, internal to the kernels
    for v, cam in enumerate(cams):
        vr = oracle.render_view(scene, cam, bg=BG, tile=tile)
        ex = excluded_pixels(vr, cam, tile=tile)
        assert np.abs(out[v].rgb.cpu().numpy() - vr.rgb)[:, ~ex].max() <= IMG_TOL
        np.testing.assert_array_equal(out[v].n_contrib.cpu().numpy()[~ex], vr.n_contrib[~ex])


def test_autotuner_marks_candidates_over_budget():
    scene, cams, dls = small_multiview(seed=7, n=3000, views=2, W=256, H=160)
    g = to_gpu(scene)
    keys16 = sum(int(oracle.keys(oracle.project(scene, c), c)[0].size) for c in cams)
    keys32 = sum(int(oracle.keys(oracle.project(scene, c, (32, 32)), c, (32, 32))[0].size) for c in cams)
    assert keys32 < keys16
    from paper_2411_14847_amd import Context
    tiles = sum(((c.width + 15) // 16) * ((c.height + 15) // 16) for c in cams)
    ctx = Context(max_gaussians=scene.n, max_views=len(cams), max_keys=keys32, max_tiles=tiles)
    ctx.tile = (32, 32)
    out = ctx.render_fwd(g, cams, BG)
    dl_t = [torch.as_tensor(d, device="cuda") for d in dls]
    res = ctx.autotune_tile(g, cams, BG, out, dl_t, g.zeros_like(), candidates=((16, 16), (32, 32)), reps=1)
    log(f"  autotune under a tight key budget: {res}")
    assert res[(16, 16)] is None and res[(32, 32)] is not None and ctx.tile == (32, 32)
    ctx.sync()


@pytest.mark.parametrize("tile", [(16, 16), (64, 32)])
def test_keys_of_views_of_different_sizes(tile):
    """Tile keys are relative to their view: views of 1352x1014 (5,440 16x16 tiles, whose ids
    take two sort passes; 352 at 64x32, one pass) batched with a 40x30 view. Keys, values and
    ranges of every view bit-exact against the oracle."""
    scene, _, _ = synth.multiview_scene(51, n=3000, n_views=1, width=1352, height=1014, with_grads=False)
    cams = synth.multiview_rig(1352, 1014)[:2] + synth.multiview_rig(40, 30)[2:3]
    log(f"[keys by view] tile {tile}, sizes {[(c.width, c.height) for c in cams]}")
    g = to_gpu(scene)
    ctx = make_ctx(scene.n, cams)
    ctx.tile = tile
    ctx.render_fwd(g, cams, BG)
    ctx.sync()
    for v, cam in enumerate(cams):
        p = oracle.project(scene, cam, tile)
        k, val, r = oracle.keys(p, cam, tile)
        TX, TY = oracle.tiles_of(cam, tile)
        gk, gv, gr = ctx.debug_keys(v, k.size + 16, TX * TY)
        assert k.size > 0
        np.testing.assert_array_equal(gk, k)
        np.testing.assert_array_equal(gv, val)
        np.testing.assert_array_equal(gr, r)


def test_backward_rejects_another_subtile_size_than_the_forwards():
    from paper_2411_14847_amd import DassError
    scene, cams, dls = small_multiview(seed=12, n=800, views=2, W=96, H=80)
    g = to_gpu(scene)
    ctx = make_ctx(scene.n, cams)
    ctx.tile = (32, 32)
    out = ctx.render_fwd(g, cams, BG)
    ctx.tile = (32, 32, 8)
    with pytest.raises(DassError, match="DASS_E_INVALID"):
        ctx.render_bwd(g, cams, BG, out, [torch.as_tensor(d, device="cuda") for d in dls], g.zeros_like())
    ctx.sync()


@pytest.mark.parametrize("n,log_scale", [(1, -2.0), (63, -4.0), (64, -1.0), (65, -4.0), (513, -4.0), (1100, -2.0)])
@pytest.mark.parametrize("tile", [(16, 16), (64, 64)])
def test_tile_lists_at_group_chunk_and_window_edges(n, log_scale, tile):
    """The binning places 64 Gaussians at a time (by key, or by tile where most rectangles cover most
    of their common box), in chunks of up to 512 and windows of at most 256 (count: 1,024) tiles: Gaussian counts
    around 64 and 512, narrow and wide footprints, views of 1,408 and 30 tiles and one 1,040 tiles
    wide.  Lists and ranges of every view bit-exact against the oracle."""
    scene, _ = synth.frustum_scene(90 + n, n, 0, log_scale, 0.5)
    cams = [synth.make_camera(np.eye(3), (0.0, 0.0, 0.0), w, h) for w, h in ((700, 500), (90, 75), (16640, 40))]
    log(f"[lists] n {n} log-scale {log_scale} tile {tile}")
    g = to_gpu(scene)
    ctx = make_ctx(scene.n, cams, keys_per_gaussian=4200)
    ctx.tile = tile
    ctx.render_fwd(g, cams, BG)
    ctx.sync()
    for v, cam in enumerate(cams):
        p = oracle.project(scene, cam, tile)
        assert not np.any(p.flags & oracle.FLAG_RADIUS)
        k, val, r = oracle.keys(p, cam, tile)
        TX, TY = oracle.tiles_of(cam, tile)
        gk, gv, gr = ctx.debug_keys(v, k.size + 16, TX * TY)
        np.testing.assert_array_equal(gk, k)
        np.testing.assert_array_equal(gv, val)
        np.testing.assert_array_equal(gr, r)


@pytest.mark.parametrize("n,mix", [(28_001, False), (32_805, False), (32_805, True)])
def test_tile_lists_of_wide_gaussians_in_long_chunks(n, mix):
    """32 views, so that a chunk holds seven or eight groups of 64: wide footprints, placed by tile eight
    groups at a time with the last ones short or missing, and (mix) wide ones among narrow ones in
    depth order, so that such a piece begins among wide and ends among narrow ones.  Lists of the
    first and the last view bit-exact against the oracle."""
    scene, _ = synth.frustum_scene(7, n, 0, -4.0, 0.3)
    z = scene.mean[2]
    wide = (np.sin(z * 40.0) > 0.0) if mix else np.ones(n, bool)
    scene.log_scale[:, wide] += 3.5
    cams = [synth.make_camera(np.eye(3), (0.0, 0.0, 0.0), 700 - 3 * v, 500 - v) for v in range(32)]
    log(f"[lists] n {n} mix {mix}")
    g = to_gpu(scene)
    ctx = make_ctx(scene.n, cams, keys_per_gaussian=90)
    ctx.tile = (64, 64)
    ctx.render_fwd(g, cams, BG)
    ctx.sync()
    for v in (0, 31):
        p = oracle.project(scene, cams[v], (64, 64))
        k, val, r = oracle.keys(p, cams[v], (64, 64))
        TX, TY = oracle.tiles_of(cams[v], (64, 64))
        log(f"  view {v}: {k.size} keys of {n} Gaussians on {TX * TY} tiles")
        gk, gv, gr = ctx.debug_keys(v, k.size + 16, TX * TY)
        np.testing.assert_array_equal(gk, k)
        np.testing.assert_array_equal(gv, val)
        np.testing.assert_array_equal(gr, r)


@pytest.mark.parametrize("make", ["opaque", "ragged"])
def test_blend_by_quadrant_matches_blend_by_subtile(make):
    """A call of few 16x16 sub-tiles is blended by one wave per 8x8 quadrant, one of many by one wave
    per sub-tile.  The same view rendered alone and three times over (few, the views' sub-tiles taken in
    turn) and eighteen times (more than 10,240 sub-tiles; 4,096 for the backward): images, T_final and
    n_contrib bit-identical; gradients of the k-fold call are k times the single one's up to the order of
    the float sums (1e-5 of the tensor's largest, the sums having a few hundred terms of 2^-24 relative
    rounding each)."""
    scene, cams, _ = (synth.opaque_scene(5, n=900, width=485, height=318, sh_degree=1) if make == "opaque"
                      else synth.tiny_scene(6, 1500, 489, 327, sh_degree=2, log_scale_mu=-2.2))
    folds = (1, 3, 18)
    rng = np.random.default_rng(9)
    dl = torch.as_tensor(rng.normal(size=(3, cams[0].height, cams[0].width)).astype(np.float32), device="cuda")
    log(f"[by quadrant] {make}")
    g = to_gpu(scene)
    res = []
    for k in folds:
        cc = cams * k
        ctx = make_ctx(scene.n, cc, keys_per_gaussian=700)
        out = ctx.render_fwd(g, cc, BG)
        grads = g.zeros_like()
        ctx.render_bwd(g, cc, BG, out, [dl] * len(cc), grads)
        ctx.sync()
        res.append((out, grads))
    for k, (out, grads) in zip(folds[1:], res[1:]):
        for o in out:
            assert torch.equal(o.rgb, res[0][0][0].rgb) and torch.equal(o.t_final, res[0][0][0].t_final)
            assert torch.equal(o.n_contrib, res[0][0][0].n_contrib)
        for a, b in zip(res[0][1].planes(), grads.planes()):
            scale = float(a.abs().max())
            assert scale > 0.0
            assert float((b / k - a).abs().max()) <= 1e-5 * scale


@pytest.mark.parametrize("n", [1, 63, 1025, 2048, 2049, 4097, 8193, 12289, 16384, 16385, 40000])
@pytest.mark.parametrize("depths", ["far", "ties", "hidden"])
def test_depth_order_at_the_sorts_edges(n, depths):
    """The depth sort holds a view of up to 16,384 Gaussians in LDS (2,048 to 16,384 slots) and sorts
    larger ones in three 9-bit digits, a fourth where a depth lies beyond 13,107: depths over
    six decades (far), a few distinct depths (ties, index order) and none visible in view 1 (hidden).
    Lists bit-exact against the oracle."""
    rng = np.random.default_rng(n)
    scene, _ = synth.frustum_scene(17 + n, n, 0, -4.0, 0.5)
    z = np.exp(rng.uniform(np.log(0.21), np.log(3e5), n)) if depths == "far" else rng.choice([2.0, 2.5, 3.0, 70.0], n)
    scene.mean[2] = z.astype(np.float32)
    scene.mean[:2] = (rng.uniform(-0.4, 0.4, (2, n)) * z).astype(np.float32)
    scene.log_scale[:] = (np.log(0.004 * z) + rng.normal(0, 0.3, (3, n))).astype(np.float32)
    cams = [synth.make_camera(np.eye(3), (0.0, 0.0, 0.0), 320, 200),
            synth.make_camera(np.diag([1.0, -1.0, -1.0]) if depths == "hidden" else np.eye(3), (0.05, 0.0, 0.0), 64, 64)]
    log(f"[depth order] n {n} {depths}")
    g = to_gpu(scene)
    ctx = make_ctx(scene.n, cams)
    for _ in range(2):  # the second call starts from what the first left behind
        ctx.render_fwd(g, cams, BG)
    ctx.sync()
    for v, cam in enumerate(cams):
        p = oracle.project(scene, cam, (16, 16))
        assert not np.any(p.flags & oracle.FLAG_RADIUS)
        k, val, r = oracle.keys(p, cam, (16, 16))
        TX, TY = oracle.tiles_of(cam, (16, 16))
        gk, gv, gr = ctx.debug_keys(v, k.size + 16, TX * TY)
        np.testing.assert_array_equal(gk, k)
        np.testing.assert_array_equal(gv, val)
        np.testing.assert_array_equal(gr, r)


def _scene_with_far_depths(n, share, top=1e10):
    """n small Gaussians at depths 2 to 10, `share` of them (at least one) at depths 13,000 to `top` instead."""
    rng = np.random.default_rng(n)
    scene, _ = synth.frustum_scene(29, n, 0, -4.0, 0.5)
    z = rng.uniform(2.0, 10.0, n)
    far = rng.choice(n, max(1, int(n * share)), replace=False)
    z[far] = np.exp(rng.uniform(np.log(1.3e4), np.log(top), far.size))
    z[far[0]] = 20_000.0
    scene.mean[2] = z.astype(np.float32)
    scene.mean[:2] = (rng.uniform(-0.4, 0.4, (2, n)) * z).astype(np.float32)
    scene.log_scale[:] = (np.log(0.002 * z) + rng.normal(0, 0.3, (3, n))).astype(np.float32)
    return scene, far


@pytest.mark.parametrize("n,views,share", [(16_385, 1, 0.0), (16_385, 3, 0.5), (60_001, 3, 0.05), (60_001, 9, 0.9)])
def test_depth_order_with_far_depths_among_near_ones(n, views, share):
    """A view with depths beyond 13,107 takes a fourth digit, spread over 8 to 32 workgroups: a single far
    Gaussian, few and most of them, over several of that digit's values, the other views without any
    (looking the other way).  Lists bit-exact against the oracle, in a second call as in the first."""
    scene, _ = _scene_with_far_depths(n, share)
    away = np.diag([1.0, -1.0, -1.0])
    cams = [synth.make_camera(away if v % 2 else np.eye(3), (0.01 * v, 0.0, 0.0), 320, 200) for v in range(views)]
    log(f"[far depths] n {n} views {views} share {share}")
    g = to_gpu(scene)
    ctx = make_ctx(scene.n, cams)
    for _ in range(2):
        ctx.render_fwd(g, cams, BG)
    ctx.sync()
    for v, cam in enumerate(cams):
        p = oracle.project(scene, cam, (16, 16))
        assert not np.any(p.flags & oracle.FLAG_RADIUS)
        k, val, r = oracle.keys(p, cam, (16, 16))
        TX, TY = oracle.tiles_of(cam, (16, 16))
        gk, gv, gr = ctx.debug_keys(v, k.size + 16, TX * TY)
        np.testing.assert_array_equal(gk, k)
        np.testing.assert_array_equal(gv, val)
        np.testing.assert_array_equal(gr, r)


def test_far_gaussians_do_not_dominate_a_views_time():
    """One Gaussian of 300k at depth 20,000, or a tenth of them: the render takes at most half as long again as
    with all near (their digit of the sort is one more pass of four; by one workgroup it took as long
    as several renders)."""
    scene, far = _scene_with_far_depths(300_000, 0.1)
    cams = [synth.make_camera(np.eye(3), (0.0, 0.0, 0.0), 640, 480)]
    ctx = make_ctx(scene.n, cams)
    out, best = None, {}
    at = np.random.default_rng(3).uniform(-0.4, 0.4, (2, far.size))
    for rep in range(6):
        for name, of in (("near", far[:0]), ("one", far[:1]), ("tenth", far)):
            z = np.full(far.size, 9.0)
            z[:of.size] = 20_000.0
            scene.mean[:, far] = np.concatenate([at * z, z[None]])
            scene.log_scale[:, far] = np.log(0.002 * z)
            g = to_gpu(scene)
            out = ctx.render_fwd(g, cams, BG, out=out)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            ctx.sync()
            a.record()
            for _ in range(10):
                ctx.render_fwd(g, cams, BG, out=out)
            b.record()
            b.synchronize()
            best[name] = min(best.get(name, 1e9), a.elapsed_time(b) / 10)
    log(f"  ms: {best}")
    assert best["one"] <= 1.5 * best["near"] and best["tenth"] <= 1.5 * best["near"]


def test_backward_of_one_wide_view_does_not_slow_down_below_its_rules_line():
    """Wide footprints, one view: the backward of 1024x1024 (4,096 sub-tiles) takes no longer than that of the
    slightly larger 1088x1024, whatever kernel either is given (it took a fifth longer by quadrants)."""
    rng = np.random.default_rng(11)
    n = 100_000
    scene, _ = synth.frustum_scene(11, n, 0, -2.0, 0.5)
    z = rng.uniform(2.0, 10.0, n)
    scene.mean[:] = np.concatenate([rng.uniform(-0.4, 0.4, (2, n)) * z, z[None]])
    g = to_gpu(scene)
    grads, ms = g.zeros_like(), {}
    for rep in range(4):
        for w in (1024, 1088):
            cams = [synth.make_camera(np.eye(3), (0.0, 0.0, 0.0), w, 1024)]
            ctx = make_ctx(n, cams, keys_per_gaussian=90)
            ctx.tile = (64, 64)
            out = ctx.render_fwd(g, cams, BG)
            dl = [torch.ones(3, 1024, w, device="cuda")]
            ctx.render_bwd(g, cams, BG, out, dl, grads)
            ctx.sync()
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                ctx.render_bwd(g, cams, BG, out, dl, grads)
            b.record()
            b.synchronize()
            ms[w] = min(ms.get(w, 1e9), a.elapsed_time(b) / 10)
    log(f"  ms by width: {ms}")
    assert ms[1024] <= 1.1 * ms[1088]


@pytest.mark.parametrize("batch", [64, 128, 256])
def test_blend_kernels_agree_in_mixed_calls_and_for_every_batch(batch):
    """A view by itself (both directions by quadrant), nine times over (5,859 sub-tiles: the forward by quadrant, the
    backward by sub-tile, as one 1352x1014 view takes it) and eighteen times (both by sub-tile), with
    every batch: images, T_final and n_contrib bit-identical, gradients as in the test above."""
    scene, cams, _ = synth.tiny_scene(6, 1500, 489, 327, sh_degree=2, log_scale_mu=-2.2)
    rng = np.random.default_rng(9)
    dl = torch.as_tensor(rng.normal(size=(3, cams[0].height, cams[0].width)).astype(np.float32), device="cuda")
    g = to_gpu(scene)
    one = None
    for k in (1, 9, 18):
        cc = cams * k
        ctx = make_ctx(scene.n, cc, keys_per_gaussian=700)
        ctx.batch = batch
        out = ctx.render_fwd(g, cc, BG)
        grads = g.zeros_like()
        ctx.render_bwd(g, cc, BG, out, [dl] * k, grads)
        ctx.sync()
        one = one or (out[0], grads)
        for o in out:
            assert torch.equal(o.rgb, one[0].rgb) and torch.equal(o.t_final, one[0].t_final)
            assert torch.equal(o.n_contrib, one[0].n_contrib)
        for a, b in zip(one[1].planes(), grads.planes()):
            scale = float(a.abs().max())
            assert scale > 0.0 and float((b / k - a).abs().max()) <= 1e-5 * scale


@pytest.mark.parametrize("of", ["colours", "pixel gradients"])
def test_infinities_spread_no_further_by_quadrant_than_by_subtile(of):
    """Gaussians of infinite colour among opaque ones, or pixel gradients that are no numbers: the same pixels and
    Gaussians get values that are no numbers whether a wave takes a quadrant, two entries at a time, or a sub-tile, one entry at a time (each pixel's
    and each entry's operations are the same, and an entry no pixel of a quadrant takes adds nothing)."""
    scene, cams, _ = synth.opaque_scene(5, n=900, width=485, height=318, sh_degree=0)
    scene.logit[::3] -= 4.0  # faint ones too, with wide margins where no pixel takes them
    rng = np.random.default_rng(9)
    dl = torch.as_tensor(rng.normal(size=(3, cams[0].height, cams[0].width)).astype(np.float32), device="cuda")
    if of == "colours":
        scene.sh[:, 5::29] = np.inf
    else:
        dl[1, 150:170:7, 200:280:9] = float("nan")
    g = to_gpu(scene)
    res = []
    for k in (1, 18):
        cc = cams * k
        ctx = make_ctx(scene.n, cc, keys_per_gaussian=700)
        out = ctx.render_fwd(g, cc, BG)
        grads = g.zeros_like()
        ctx.render_bwd(g, cc, BG, out, [dl] * k, grads)
        ctx.sync()
        res.append((out[0], grads))
    (a, ga), (b, gb) = res
    bad = ~torch.isfinite(a.rgb)
    log(f"  pixels that are no numbers: {int(bad.any(0).sum())} of {bad[0].numel()}, by sub-tile "
        f"{int((~torch.isfinite(b.rgb)).any(0).sum())}")
    log(f"  gradients: {[int((~torch.isfinite(p)).sum()) for p in ga.planes()]}, by sub-tile "
        f"{[int((~torch.isfinite(p)).sum()) for p in gb.planes()]} of {[p.numel() for p in ga.planes()]}")
    assert int(bad.sum()) < bad.numel() and (int(bad.sum()) > 0) == (of == "colours")
    same = torch.equal(torch.nan_to_num(a.rgb, 7.0), torch.nan_to_num(b.rgb, 7.0))
    assert same
    for p, q in zip(ga.planes(), gb.planes()):
        same = torch.equal(torch.isfinite(p), torch.isfinite(q))
        assert same


def test_a_context_for_very_many_tiles_stays_small():
    """max_tiles of 2^26: beside 12 bytes per tile (ranges, totals) the binning's histogram takes 1 GB, not 128
    counts per tile (34 GB), and a render in such a context is the same as in one made to measure."""
    from paper_2411_14847_amd import Context
    scene, cams, _ = synth.tiny_scene(6, 1500, 489, 327, sh_degree=0, log_scale_mu=-2.2)
    g = to_gpu(scene)
    small = make_ctx(scene.n, cams, keys_per_gaussian=700)
    want = small.render_fwd(g, cams, BG)[0]
    small.sync()
    free, _ = torch.cuda.mem_get_info()
    ctx = Context(max_gaussians=scene.n, max_views=1, max_keys=700 * scene.n, max_tiles=1 << 26)
    took = free - torch.cuda.mem_get_info()[0]
    log(f"  context for 2^26 tiles: {took / 2**30:.2f} GB")
    got = ctx.render_fwd(g, cams, BG)[0]
    ctx.sync()
    assert torch.equal(got.rgb, want.rgb) and torch.equal(got.n_contrib, want.n_contrib)
    assert took < 3 << 30


@pytest.mark.parametrize("n", [63, 319, 321, 1500])
@pytest.mark.parametrize("log_scale", [-4.0, -1.5])
def test_tile_lists_in_chunks_set_by_the_views_tiles(n, log_scale):
    """Views of 17,672 tiles take 320 Gaussians to a chunk whatever their number (69 windows): lists and
    ranges of narrow and wide footprints bit-exact against the oracle."""
    scene, _ = synth.frustum_scene(70 + n, n, 0, log_scale, 0.5)
    cams = [synth.make_camera(np.eye(3), (0.02 * v, 0.0, 0.0), 3000, 1500) for v in range(2)]
    g = to_gpu(scene)
    ctx = make_ctx(scene.n, cams, keys_per_gaussian=17_700)
    ctx.render_fwd(g, cams, BG)
    ctx.sync()
    for v, cam in enumerate(cams):
        p = oracle.project(scene, cam, (16, 16))
        assert not np.any(p.flags & oracle.FLAG_RADIUS)
        k, val, r = oracle.keys(p, cam, (16, 16))
        TX, TY = oracle.tiles_of(cam, (16, 16))
        log(f"[lists] n {n} log-scale {log_scale} view {v}: {k.size} keys on {TX * TY} tiles")
        gk, gv, gr = ctx.debug_keys(v, k.size + 16, TX * TY)
        np.testing.assert_array_equal(gk, k)
        np.testing.assert_array_equal(gv, val)
        np.testing.assert_array_equal(gr, r)
