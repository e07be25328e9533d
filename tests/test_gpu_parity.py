"""GPU parity: the HIP path through the C ABI against the FP64 oracle."""
import math
import sys

import numpy as np
import pytest
import torch

import scenegen
from oracle import render4d as O
from tests import parity as PT

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _np(t):
    return t.detach().cpu().numpy()


def _render_one(r, cam, t):
    rgb, dep, alp = r.render([cam], [t])
    torch.cuda.synchronize()
    h, w = cam.height, cam.width
    return _np(rgb).reshape(3, h, w), _np(dep).reshape(h, w), _np(alp).reshape(h, w)


def _needle_scene(seed, n, grow, shrink):
    """Footprints stretched along one axis (log scale + grow) and thinned
    along the others (- shrink), at random orientations."""
    sc = scenegen.random_scene(seed, n, sh_degree=1, t_order=1, mu_log_t=-1.0)
    sc.log_scales4[:, 0] += np.float32(grow)
    sc.log_scales4[:, 1:3] -= np.float32(shrink)
    return sc


def _big_splat_scene(seed, n, grow=1.0, spread=1.0, sh=2, to=2, mu_log_t=-1.5):
    sc = scenegen.random_scene(seed, n, sh_degree=sh, t_order=to, spread=spread, mu_log_t=mu_log_t)
    sc.log_scales4[:, :3] += np.float32(grow)
    return sc


CASES = [
    # name, scene factory, camera, t, bg
    ("cfg0", lambda: scenegen.make_workload(0).scene, lambda: scenegen.make_workload(0).cameras[0], 0.5,
     (0.0, 0.0, 0.0)),
    ("ragged_100x70", lambda: _big_splat_scene(5, 3000, grow=0.8),
     lambda: scenegen.look_at_camera((1.0, 0.5, 3.5), 100, 70), 0.37, (0.2, 0.1, 0.05)),
    ("dense_stop_48x40", lambda: _big_splat_scene(6, 2500, grow=1.5, spread=0.5, sh=3, to=1),
     lambda: scenegen.look_at_camera((0.0, -0.3, 3.0), 48, 40), 0.6, (0.0, 0.0, 0.0)),
    # needle-like footprints at every orientation: the per-quadrant ellipse
    # test that decides which entries a wave walks is at its tightest here
    ("needles_90x66", lambda: _needle_scene(9, 2000, 1.2, 0.8),
     lambda: scenegen.look_at_camera((0.4, 0.2, 3.2), 90, 66), 0.45, (0.1, 0.2, 0.3)),
]


@pytest.mark.parametrize("name,mk_scene,mk_cam,t,bg", CASES, ids=[c[0] for c in CASES])
def test_forward_image_parity(name, mk_scene, mk_cam, t, bg):
    _say(f"[forward parity] {name}")
    scene, cam = mk_scene(), mk_cam()
    r, _ = PT.gpu_setup(scene, bg)
    g_rgb, g_dep, g_alp = _render_one(r, cam, t)
    out, img = PT.oracle_view(scene, cam, t, bg)
    res = PT.compare_images(g_rgb, g_dep, g_alp, img)
    _say(f"  {res}")
    # per-pixel backward state: the last contributor is the same primitive
    # away from flagged pixels, and the final transmittance agrees
    ok = ~img["unc"].numpy()
    ok_order = ok & ~img["unc_o"].numpy()        # an FP32 depth tie may reorder the last pair
    g_last = PT.last_contributor_ids(r, cam, r.debug("ids").astype(np.int64))
    o_last = PT.oracle_last_ids(out, cam)
    assert (g_last[ok_order] == o_last[ok_order]).all()
    T = r.debug("pix_t").reshape(cam.height, cam.width)
    assert np.allclose(T[ok], img["T"].numpy()[ok], atol=2e-5)


@pytest.mark.parametrize("name,mk_scene,mk_cam,t,bg", CASES, ids=[c[0] for c in CASES])
def test_preprocess_records_parity(name, mk_scene, mk_cam, t, bg):
    """The forward geometry is evaluated in FP64 and rounded once: every
    record value (u, v, z, conic, opacity * p(t)) equals the oracle's FP64
    value rounded to float32, bit for bit (a value within 1e-10 of a rounding
    midpoint may take the other neighbour); the colour (a float32 4DSH sum)
    is within 2e-6. The active set is the oracle's minus the primitives
    that cannot reach alpha 1/255 anywhere in their rectangle (the default
    binning culls those), and each rectangle is the oracle's 3-sigma
    rectangle cut to the alpha-floor box."""
    _say(f"[preprocess parity] {name}")
    scene, cam = mk_scene(), mk_cam()
    r, _ = PT.gpu_setup(scene, bg)
    r.render([cam], [t])
    recs, ids = r.debug("records"), r.debug("ids")
    pre = O.preprocess(O.params_from_scene(scene), O.to_ocamera(cam), PT.f32(t), scene.sh_degree, scene.t_order,
                       scene.t_period)
    act_o = pre["active"].numpy()
    rs, rm = pre["rect_sure"].numpy(), pre["rect_maybe"].numpy()
    area = lambda rr: np.maximum(rr[:, 2] - rr[:, 0], 0) * np.maximum(rr[:, 3] - rr[:, 1], 0)
    unsure = (area(rs) == 0) & (area(rm) > 0)
    act_g = np.zeros(scene.n, bool)
    act_g[ids] = True
    tight, visible = PT.alpha_floor_box(pre, cam)
    assert not (act_g & ~act_o & ~unsure).any(), np.nonzero(act_g & ~act_o & ~unsure)[0][:10]
    dropped = act_o & ~act_g & ~unsure
    assert not (dropped & visible).any(), np.nonzero(dropped & visible)[0][:10]
    common = ids[act_o[ids]]
    row = {int(g): i for i, g in enumerate(ids)}
    sel = np.array([row[int(g)] for g in common])
    R = recs[sel]
    doubt = pre["rec_doubt"].numpy()[common]
    f32 = lambda k: pre[k].numpy()[common].astype(np.float32)
    for col, key in ((0, "u32"), (1, "v32"), (2, "z32"), (3, "opac32")):
        same = R[:, col] == f32(key)
        assert (same | doubt).all(), (key, int((~same & ~doubt).sum()))
    same = R[:, 4:7] == pre["conic32"].numpy()[common].astype(np.float32)
    assert (same.all(1) | doubt).all(), int((~same.all(1) & ~doubt).sum())
    _say(f"  {len(common)} records bit-exact ({int(doubt.sum())} with a rounding in doubt)")
    col = pre["color"].detach().numpy()[common]
    assert np.allclose(R[:, 8:11], col, atol=2e-6, rtol=0)
    rx = R[:, 7].view(np.uint32)
    ry = R[:, 11].view(np.uint32)
    rect_g = np.stack([rx & 0xFFFF, ry & 0xFFFF, rx >> 16, ry >> 16], 1).astype(np.int64)
    rect_o = pre["rect"].numpy()[common]
    edge_unsure = (rs[common] != rm[common]).any(1)
    # footprint within the 3-sigma rectangle, and covering the alpha-floor box
    inside = (rect_g[:, :2] >= rect_o[:, :2]).all(1) & (rect_g[:, 2:] <= rect_o[:, 2:]).all(1)
    assert (inside | edge_unsure).all()
    tt = tight[common]
    vis = visible[common]
    covers = (rect_g[:, :2] <= tt[:, :2]).all(1) & (rect_g[:, 2:] >= tt[:, 2:]).all(1)
    assert (covers | ~vis | edge_unsure).all()
    # depth order: non-decreasing float z, ties by (view, index)
    zg = recs[:, 2]
    assert (np.diff(zg) >= 0).all()
    tie = np.diff(zg) == 0
    assert (np.diff(ids.astype(np.int64))[tie] > 0).all()


BIG_CASES = [
    # footprints taller than 256 px: blocks of 64 records span more than 1024
    # tile rows (the emission's per-instance row walk)
    ("big_splats_1352x1014", lambda: _big_splat_scene(41, 600, grow=1.9, sh=1, to=1),
     lambda: scenegen.look_at_camera((0.3, 0.2, 3.3), 1352, 1014), 0.5, (0.0, 0.0, 0.0)),
    # medium footprints: some blocks of 64 records hold more than 4096
    # instances in at most 1024 rows (the emission's chunked instance map)
    ("medium_splats_1352x1014", lambda: _big_splat_scene(42, 3000, grow=0.3, sh=1, to=1),
     lambda: scenegen.look_at_camera((0.3, 0.2, 3.5), 1352, 1014), 0.5, (0.0, 0.0, 0.0)),
]
REF_CASES = CASES + BIG_CASES


def _emit_blocks(recs):
    """Per block of 64 depth-ordered records (one emission workgroup): tile
    rows and instances of the records' rectangles."""
    rx, ry = recs[:, 7].view(np.uint32), recs[:, 11].view(np.uint32)
    rows = (ry >> 16).astype(np.int64) - (ry & 0xFFFF)
    cols = (rx >> 16).astype(np.int64) - (rx & 0xFFFF)
    br = np.array([rows[i:i + 64].sum() for i in range(0, len(rows), 64)], np.int64)
    bi = np.array([(rows * cols)[i:i + 64].sum() for i in range(0, len(rows), 64)], np.int64)
    return br, bi


@pytest.mark.parametrize("name,mk_scene,mk_cam,t,bg", REF_CASES, ids=[c[0] for c in REF_CASES])
def test_reference_footprint_tile_lists_bit_exact(name, mk_scene, mk_cam, t, bg):
    """With G4D_TUNE_ELLIPSE_CULL = 0 the library bins by the plain
    footprint rule of the definition: the active set, every record's 3-sigma
    tile rectangle and therefore the instance count equal the oracle's, and
    every tile's sorted list equals the oracle's list of the primitives whose
    rectangle covers it, ordered by (float32 depth, index) -- the order of the
    identical float32 keys. Primitives with a decision within the FP64 margin
    (p(t), near plane, radius or rectangle edge) are left out of the
    comparison and counted (expected: none or a few)."""
    _say(f"[reference footprint] {name}")
    from paper_2310_10642_amd import g4d
    scene, cam = mk_scene(), mk_cam()
    r, _ = PT.gpu_setup(scene, bg)
    r.set_tuning(g4d.G4D_TUNE_ELLIPSE_CULL, 0)
    rgb, dep, alp = r.render([cam], [t])
    torch.cuda.synchronize()
    recs, ids = r.debug("records"), r.debug("ids").astype(np.int64)
    vals, ranges = r.debug("tile_vals"), r.debug("ranges")
    stats = r.stats()
    pre = O.preprocess(O.params_from_scene(scene), O.to_ocamera(cam), PT.f32(t), scene.sh_degree, scene.t_order,
                       scene.t_period)
    act_o = pre["active"].numpy()
    rs, rm = pre["rect_sure"].numpy(), pre["rect_maybe"].numpy()
    doubtful = (rs != rm).any(1)
    act_g = np.zeros(scene.n, bool)
    act_g[ids] = True
    assert ((act_g == act_o) | doubtful).all(), np.nonzero((act_g != act_o) & ~doubtful)[0][:10]
    rx, ry = recs[:, 7].view(np.uint32), recs[:, 11].view(np.uint32)
    rect_g = np.stack([rx & 0xFFFF, ry & 0xFFFF, rx >> 16, ry >> 16], 1).astype(np.int64)
    rect_o = pre["rect"].numpy()[ids]
    ok = ~doubtful[ids]
    assert (rect_g[ok] == rect_o[ok]).all()
    area = (rect_g[:, 2] - rect_g[:, 0]) * (rect_g[:, 3] - rect_g[:, 1])
    assert stats["instances"] == int(area.sum())
    br, bi = _emit_blocks(recs)
    _say(f"  {len(ids)} records, {stats['instances']} instances, {int(doubtful[act_o | act_g].sum())} in doubt; "
         f"emission blocks over 1024 rows: {int((br > 1024).sum())}, chunked (> 4096 instances): "
         f"{int(((br <= 1024) & (bi > 4096)).sum())}")
    if name == "big_splats_1352x1014":
        assert (br > 1024).any()
    if name == "medium_splats_1352x1014":
        assert ((br <= 1024) & (bi > 4096)).any()
    # per-tile lists: the oracle's primitives covering the tile by (float32 z, index)
    z32 = pre["z32"].numpy().astype(np.float32)
    skip = set(np.nonzero(doubtful)[0].tolist())
    tx = (cam.width + 15) // 16
    rect_all = pre["rect"].numpy()
    act_idx = np.nonzero(act_o & ~doubtful)[0]
    order = act_idx[np.lexsort((act_idx, z32[act_idx]))]
    ro = rect_all[order]
    for tid in range(ranges.shape[0]):
        txi, tyi = tid % tx, tid // tx
        cov = (ro[:, 0] <= txi) & (txi < ro[:, 2]) & (ro[:, 1] <= tyi) & (tyi < ro[:, 3])
        want = order[cov]
        s0, e0 = ranges[tid]
        got = [int(g) for g in ids[vals[s0:e0]] if int(g) not in skip]
        assert got == want.tolist(), (tid, got[:8], want[:8].tolist())
    # and the images are those of the default binning
    r.set_tuning(g4d.G4D_TUNE_ELLIPSE_CULL, 1)
    rgb1, dep1, alp1 = r.render([cam], [t])
    assert torch.equal(rgb, rgb1) and torch.equal(dep, dep1) and torch.equal(alp, alp1)


def _box_min_q(a, b, c, ex0, ex1, ey0, ey1):
    """FP64 minimum of a dx^2 + 2 b dx dy + c dy^2 over [ex0, ex1] x [ey0, ey1]
    (a convex quadratic: 0 when the box holds the origin, else the smallest
    of the four edges' clamped 1D minima)."""
    q = lambda dx, dy: a * dx * dx + 2 * b * dx * dy + c * dy * dy
    cands = [q(ex, np.clip(-b * ex / c, ey0, ey1)) for ex in (ex0, ex1)]
    cands += [q(np.clip(-b * ey / a, ex0, ex1), ey) for ey in (ey0, ey1)]
    inside = (ex0 <= 0) & (ex1 >= 0) & (ey0 <= 0) & (ey1 >= 0)
    return np.where(inside, 0.0, np.minimum.reduce(cands))


@pytest.mark.parametrize("name,mk_scene,mk_cam,t,bg", REF_CASES, ids=[c[0] for c in REF_CASES])
def test_binning_is_a_valid_stable_sort(name, mk_scene, mk_cam, t, bg):
    """The (tile, record) instances are ordered by tile then by depth position
    and delimited by the tile ranges; each record is listed in the tiles of
    its rectangle that its alpha-floor ellipse reaches: every tile whose
    pixel-centre box meets Q <= 2 ln(255 opacity) (FP64, on the stored FP32
    record) is there, none well beyond it (0.1 % + 0.02 and 0.01 px are the
    kernel's slack; the bound here allows 1 % + 0.5)."""
    _say(f"[binning] {name}")
    scene, cam = mk_scene(), mk_cam()
    r, _ = PT.gpu_setup(scene, bg)
    r.render([cam], [t])
    recs = r.debug("records").astype(np.float64)
    keys, vals, ranges = r.debug("tile_keys"), r.debug("tile_vals"), r.debug("ranges")
    tx = (cam.width + 15) // 16
    rx, ry = r.debug("records")[:, 7].view(np.uint32), r.debug("records")[:, 11].view(np.uint32)
    got = list(zip(keys.tolist(), vals.tolist()))
    assert got == sorted(set(got))                      # by tile, then record; no duplicates
    got_set = set(got)
    must, may = set(), set()
    for d in range(recs.shape[0]):
        x0, x1, y0, y1 = int(rx[d] & 0xFFFF), int(rx[d] >> 16), int(ry[d] & 0xFFFF), int(ry[d] >> 16)
        u, v, op, a, b, c = recs[d, 0], recs[d, 1], recs[d, 3], recs[d, 4], recs[d, 5], recs[d, 6]
        L0 = 2.0 * math.log(255.0 * op)
        yy, xx = np.meshgrid(np.arange(y0, y1), np.arange(x0, x1), indexing="ij")
        qmin = _box_min_q(a, b, c, 16.0 * xx + 0.5 - u, 16.0 * xx + 15.5 - u, 16.0 * yy + 0.5 - v,
                          16.0 * yy + 15.5 - v)
        for tile, qm in zip((yy * tx + xx).ravel().tolist(), qmin.ravel().tolist()):
            if qm <= L0:
                must.add((tile, d))
            if qm <= 1.01 * L0 + 0.5:
                may.add((tile, d))
    assert must <= got_set, sorted(must - got_set)[:10]
    assert got_set <= may, sorted(got_set - may)[:10]
    # the ranges (keys are read back as the tile whose range covers them)
    # cover every instance once, in tile order
    assert (keys != 0xFFFFFFFF).all()
    assert int((ranges[:, 1].astype(np.int64) - ranges[:, 0]).clip(min=0).sum()) == len(keys)
    for tid in range(ranges.shape[0]):
        s, e = ranges[tid]
        assert e >= s
        if e > s:
            assert (keys[s:e] == tid).all()
            assert s == 0 or keys[s - 1] != tid
            assert e == len(keys) or keys[e] != tid
    stats = r.stats()
    assert stats["instances"] == len(got)
    assert stats["active_total"] == recs.shape[0]
    br, bi = _emit_blocks(r.debug("records"))
    _say(f"  instances {len(got)}: {len(must)} required, {len(may)} allowed; emission blocks over 1024 rows: "
         f"{int((br > 1024).sum())}, with more than 4096 instances: {int((bi > 4096).sum())}")


@pytest.mark.parametrize("name,mk_scene,mk_cam,t,bg", CASES, ids=[c[0] for c in CASES])
def test_backward_gradient_parity(name, mk_scene, mk_cam, t, bg):
    _say(f"[backward parity] {name}")
    scene, cam = mk_scene(), mk_cam()
    r, _ = PT.gpu_setup(scene, bg)
    r.render([cam], [t])
    out, img = PT.oracle_view(scene, cam, t, bg, requires_grad=True)
    mask = (~img["unc_g"].numpy()).astype(np.float64)
    drgb, ddep, dalp = PT.dl_maps(11, cam.height, cam.width, mask)
    L = O.tile_linear_loss(out, torch.as_tensor(drgb), torch.as_tensor(ddep), torch.as_tensor(dalp), cam)
    L.backward()
    f32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    g = r.backward(f32(drgb).reshape(-1), f32(ddep).reshape(-1), f32(dalp).reshape(-1))
    torch.cuda.synchronize()
    rep = {}
    PT.compare_grads(g, out["params"], report=rep)
    _say(f"  rel L2 {rep}")


def test_batched_equals_per_view():
    """One batched call over views of different sizes and times gives the
    per-view images bit for bit and the sum of the per-view gradients."""
    _say("[batched == per-view]")
    scene = _big_splat_scene(7, 4000, grow=0.7, sh=3, to=2)
    cams = [scenegen.look_at_camera((math.sin(a) * 3.5, 0.3, math.cos(a) * 3.5), w, h)
            for a, (w, h) in zip([0.0, 1.2, 2.5], [(64, 48), (80, 80), (33, 17)])]
    times = [0.2, 0.5, 0.85]
    r, _ = PT.gpu_setup(scene)
    rgb_b, dep_b, alp_b = r.render(cams, times)
    views_b = [[_np(x) for x in item] for item in r.split(rgb_b, dep_b, alp_b)]
    rng = np.random.default_rng(3)
    dl = [rng.normal(size=(3, c.height, c.width)).astype(np.float32) for c in cams]
    gb = r.backward(torch.from_numpy(np.concatenate([d.reshape(-1) for d in dl])).cuda())
    gsum = [torch.zeros_like(x) for x in gb]
    for v, (c, t) in enumerate(zip(cams, times)):
        rgb, dep, alp = r.render([c], [t])
        assert np.array_equal(_np(rgb).reshape(3, c.height, c.width), views_b[v][0])
        assert np.array_equal(_np(dep).reshape(c.height, c.width), views_b[v][1])
        assert np.array_equal(_np(alp).reshape(c.height, c.width), views_b[v][2])
        g = r.backward(torch.from_numpy(dl[v].reshape(-1)).cuda())
        for a, b in zip(gsum, g):
            a += b
    torch.cuda.synchronize()
    for name, a, b in zip(PT.GROUPS, gb, gsum):
        a, b = _np(a).astype(np.float64), _np(b).astype(np.float64)
        nb = np.linalg.norm(b)
        assert nb == 0 or np.linalg.norm(a - b) <= 1e-5 * nb, name


def test_round_tile_cap():
    """Thirteen 1352x1014 views (70 720 tiles) take two rounds under the
    2^16-tile cap that keeps the instance sort at two passes; every view equals
    its own single-view render bit for bit and the gradients sum."""
    _say("[round tile cap, 300k x 13 views]")
    wl = scenegen.bench_workload(13)
    r, _ = PT.gpu_setup(wl.scene)
    times = [float(x) for x in wl.times]
    rgb_b, _, _ = r.render(wl.cameras, times, depth=False, alpha=False)
    s = r.stats()
    _say(f"  rounds {s['rounds']}, tiles {s['tiles']}")
    assert s["rounds"] == 2 and s["tiles"] == 13 * 5440
    views_b = [_np(x[0]) for x in r.split(rgb_b, None, None)]
    rng = np.random.default_rng(13)
    dl = rng.uniform(-1, 1, rgb_b.numel()).astype(np.float32)
    gb = [x.clone() for x in r.backward(torch.from_numpy(dl).cuda())]
    gsum = [torch.zeros_like(x) for x in gb]
    o = 0
    for v, (c, t) in enumerate(zip(wl.cameras, times)):
        rgb, _, _ = r.render([c], [t], depth=False, alpha=False)
        assert np.array_equal(_np(rgb).reshape(views_b[v].shape), views_b[v]), v
        n = 3 * c.width * c.height
        g = r.backward(torch.from_numpy(dl[o:o + n]).cuda())
        o += n
        for a, b in zip(gsum, g):
            a += b
    _close_grads(gb, gsum)


def test_single_view_beyond_16_bit_tile_ids():
    """One 4128x4112 view has 66 306 tiles: its round's tile ids need 17 bits,
    so the instance sort takes its 32-bit-key path (three passes) instead of
    the 16-bit one every smaller round uses. The lists are a stable sort by
    (tile, depth position) and sampled tiles match the oracle."""
    _say("[one view of 66 306 tiles, 32-bit instance keys]")
    scene = scenegen.random_scene(31, 20000, sh_degree=2, t_order=1, spread=1.2)
    cam = scenegen.look_at_camera((0.0, 0.3, 3.5), 4128, 4112)
    r, _ = PT.gpu_setup(scene)
    rgb, dep, alp = r.render([cam], [0.45])
    stats = r.stats()
    _say(f"  rounds {stats['rounds']}, tiles {stats['tiles']}, instances {stats['instances']}")
    assert stats["rounds"] == 1 and stats["tiles"] == 258 * 257 > 1 << 16
    keys = r.debug("tile_keys").astype(np.int64)
    vals = r.debug("tile_vals").astype(np.int64)
    assert len(keys) == stats["instances"] > 0
    assert keys.max() >= 1 << 16  # ids past 16 bits did occur
    step = (keys[1:] > keys[:-1]) | ((keys[1:] == keys[:-1]) & (vals[1:] > vals[:-1]))
    assert step.all()
    tiles = scenegen.sample_pixels_dlddi(32, [cam], 8)[0]
    # half of the samples from the tiles past id 2^16
    far = np.arange(1 << 16, 258 * 257)
    tiles = np.concatenate([tiles[:4], np.random.default_rng(33).choice(far, 4, replace=False)]).tolist()
    _, img = PT.oracle_view(scene, cam, 0.45, tiles=tiles)
    res = PT.compare_images(_np(rgb).reshape(3, cam.height, cam.width), _np(dep).reshape(cam.height, cam.width),
                            _np(alp).reshape(cam.height, cam.width), img)
    _say(f"  tiles {tiles}: {res}")


def test_sync_free_rounds_and_graph():
    """A sync-free render of thirteen full-size views plans its two rounds
    from the tile cap alone: images, per-view counts and totals equal the
    synchronous render's, its backward (which bins the first round again
    without host reads) gives the same gradients, and the whole step
    captured into a HIP graph replays it."""
    _say("[sync-free rounds, 300k x 13 views]")
    from paper_2310_10642_amd import g4d
    wl = scenegen.bench_workload(13)
    r, _ = PT.gpu_setup(wl.scene)
    times = [float(x) for x in wl.times]
    P = sum(c.width * c.height for c in wl.cameras)
    rng = np.random.default_rng(31)
    dl = torch.from_numpy(rng.uniform(-1, 1, 3 * P).astype(np.float32)).cuda()
    ref = [x.clone() for x in r.render(wl.cameras, times)]
    s_ref = r.stats()
    g_ref = [x.clone() for x in r.backward(dl)]
    assert s_ref["rounds"] == 2
    r.set_tuning(g4d.G4D_TUNE_SYNC_FREE, 1)
    try:
        outs = (torch.empty_like(ref[0]), torch.empty_like(ref[1]), torch.empty_like(ref[2]))
        grads = r.grad_buffers()

        def step():
            r.render(wl.cameras, times, out=outs)
            r.backward(dl, out=grads)

        step()
        torch.cuda.synchronize()
        s_sf = r.stats()
        for a, b in zip(ref, outs):
            assert torch.equal(a, b)
        for k in ("rounds", "active_total", "instances", "fragments", "max_tile_list", "active_per_view"):
            assert s_ref[k] == s_sf[k], k
        _close_grads(grads, g_ref)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            step()
        for rep in range(2):
            for t in (*outs, *grads):
                t.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            for a, b in zip(ref, outs):
                assert torch.equal(a, b), rep
            _close_grads(grads, g_ref)
            _say(f"  replay {rep} ok")
        del graph
        assert r.stats()["instances"] == s_ref["instances"]
    finally:
        r.set_tuning(g4d.G4D_TUNE_SYNC_FREE, 0)


def test_autograd_function():
    """g4d.render through torch.autograd: the parameters' .grad equal the
    library's backward for the same output gradients (rgb, depth, alpha of two
    views); a central difference along the colour coefficients, which enter
    the image linearly inside the clamp, matches the directional derivative;
    and a render in between makes the pending backward an error."""
    _say("[autograd function]")
    from paper_2310_10642_amd import g4d
    scene = _big_splat_scene(11, 3000, grow=0.6, sh=3, to=2)
    # colours kept well above the clamp at 0, where the image is not smooth in the coefficients
    scene.coeffs[:, 0, :] += np.float32(1.5)
    cams = [scenegen.look_at_camera((0.5, 0.3, 3.4), 72, 56), scenegen.look_at_camera((-1.0, 0.2, 3.3), 48, 64)]
    times = [0.3, 0.7]
    r = g4d.Renderer(scene.sh_degree, scene.t_order, scene.t_period)
    leaves = [torch.from_numpy(np.ascontiguousarray(a)).cuda().requires_grad_(True)
              for a in (scene.means4, scene.log_scales4, scene.q_left, scene.q_right, scene.opacity_logit,
                        scene.coeffs)]
    rgb, dep, alp = g4d.render(r, cams, times, *leaves)
    rng = np.random.default_rng(21)
    w = [torch.from_numpy(rng.uniform(-1, 1, t.numel()).astype(np.float32)).cuda() for t in (rgb, dep, alp)]
    ((rgb * w[0]).sum() + (dep * w[1]).sum() + (alp * w[2]).sum()).backward()
    direct = [x.clone() for x in r.backward(*w)]
    _close_grads([x.grad for x in leaves], direct)
    # directional derivative along the coefficients
    d = torch.from_numpy(rng.normal(size=scene.coeffs.shape).astype(np.float32)).cuda()
    eps = 2e-4

    def f(coeffs):
        with torch.no_grad():
            o = g4d.render(r, cams, times, *leaves[:5], coeffs)
            return float(sum((t.double() * wt.double()).sum() for t, wt in zip(o, w)))

    fd = (f(leaves[5].detach() + eps * d) - f(leaves[5].detach() - eps * d)) / (2 * eps)
    an = float((leaves[5].grad.double() * d.double()).sum())
    _say(f"  directional derivative: analytic {an:.6g}, central difference {fd:.6g}")
    assert abs(fd - an) <= 1e-2 * abs(an) + 1e-3
    rgb2, _, _ = g4d.render(r, cams, times, *leaves)
    g4d.render(r, cams, times, *leaves)
    with pytest.raises(RuntimeError):
        rgb2.sum().backward()


def test_empty_and_degenerate_inputs():
    _say("[edge cases]")
    bg = (0.25, 0.5, 0.75)
    # n = 0: background everywhere
    sc = scenegen.random_scene(1, 4)
    empty = scenegen.Scene(sc.means4[:0].copy(), sc.log_scales4[:0].copy(), sc.q_left[:0].copy(),
                           sc.q_right[:0].copy(), sc.opacity_logit[:0].copy(), sc.coeffs[:0].copy(), 1, 1)
    r, _ = PT.gpu_setup(empty, bg)
    cam = scenegen.look_at_camera((0.0, 0.0, 4.0), 23, 9)
    rgb, dep, alp = _render_one(r, cam, 0.5)
    assert np.allclose(rgb, np.array(bg, np.float32)[:, None, None]) and (dep == 0).all() and (alp == 0).all()
    g = r.backward(torch.ones(3 * 23 * 9, device="cuda"))
    assert all(x.numel() == 0 for x in g)
    # every primitive culled by the temporal filter: background, zero gradients
    sc = scenegen.random_scene(2, 200, mu_log_t=-4.0)
    sc.means4[:, 3] = 0.0
    r, _ = PT.gpu_setup(sc, bg)
    rgb, dep, alp = _render_one(r, cam, 1.0)
    assert np.allclose(rgb, np.array(bg, np.float32)[:, None, None]) and r.stats()["active_total"] == 0
    g = r.backward(torch.ones(3 * 23 * 9, device="cuda"))
    assert all(float(x.abs().max()) == 0.0 for x in g)
    # 1x1 image, primitives behind the camera and at the near plane
    sc = scenegen.random_scene(3, 300, spread=2.5)
    cam1 = scenegen.look_at_camera((0.0, 0.0, 2.0), 1, 1)
    r, _ = PT.gpu_setup(sc, bg)
    g_rgb, g_dep, g_alp = _render_one(r, cam1, 0.5)
    _, img = PT.oracle_view(sc, cam1, 0.5, bg)
    PT.compare_images(g_rgb, g_dep, g_alp, img, max_flag_frac=1.0)


def test_abi_errors():
    _say("[abi errors]")
    from paper_2310_10642_amd import g4d
    r = g4d.Renderer(1, 1)
    cam = scenegen.look_at_camera((0.0, 0.0, 4.0), 8, 8)
    with pytest.raises(g4d.G4DError) as e:
        r.render([cam], [0.5])
    assert e.value.status == g4d.G4D_ESTATE
    sc = scenegen.random_scene(4, 10)
    r, _ = PT.gpu_setup(sc)
    with pytest.raises(g4d.G4DError) as e:
        r.backward(torch.zeros(192, device="cuda"))
    assert e.value.status == g4d.G4D_ESTATE
    bad = scenegen.look_at_camera((0.0, 0.0, 4.0), 8, 8)
    bad.fx = -1.0
    with pytest.raises(g4d.G4DError) as e:
        r.render([bad], [0.5])
    assert e.value.status == g4d.G4D_EINVAL
    with pytest.raises(g4d.G4DError) as e:
        r.render([cam], [float("nan")])
    assert e.value.status == g4d.G4D_EINVAL
    with pytest.raises(g4d.G4DError) as e:
        r.set_tuning(99, 1)
    assert e.value.status == g4d.G4D_EINVAL


def _sampled_parity(wl, view, n_tiles, seed, dl_seed):
    """Full-size render on the GPU; the oracle renders `n_tiles` random tiles
    of one view; images compared there, gradients for dL/dI supported there."""
    cam, t = wl.cameras[view], float(wl.times[view])
    tiles = scenegen.sample_pixels_dlddi(seed, [cam], n_tiles)[0].tolist()
    _say(f"  oracle on tiles {tiles}")
    out, img = PT.oracle_view(wl.scene, cam, t, tiles=tiles, requires_grad=True)
    r, _ = PT.gpu_setup(wl.scene)
    V = len(wl.cameras)
    rgb, dep, alp = r.render(wl.cameras, [float(x) for x in wl.times])
    item = r.split(rgb, dep, alp)[view]
    g_rgb, g_dep, g_alp = (_np(x) for x in item)
    res = PT.compare_images(g_rgb, g_dep, g_alp, img)
    _say(f"  image {res}")
    rendered = ~np.isnan(img["depth"].detach().numpy())
    mask = (rendered & ~img["unc_g"].numpy()).astype(np.float64)
    drgb, ddep, dalp = PT.dl_maps(dl_seed, cam.height, cam.width, mask)
    L = O.tile_linear_loss(out, torch.as_tensor(drgb), torch.as_tensor(ddep), torch.as_tensor(dalp), cam)
    L.backward()
    full_rgb = [np.zeros((3, c.height, c.width), np.float32) for c in wl.cameras]
    full_dep = [np.zeros((c.height, c.width), np.float32) for c in wl.cameras]
    full_alp = [np.zeros((c.height, c.width), np.float32) for c in wl.cameras]
    full_rgb[view], full_dep[view], full_alp[view] = drgb, ddep, dalp
    cat = lambda xs: torch.from_numpy(np.concatenate([x.reshape(-1) for x in xs]).astype(np.float32)).cuda()
    g = r.backward(cat(full_rgb), cat(full_dep), cat(full_alp))
    torch.cuda.synchronize()
    rep = {}
    PT.compare_grads(g, out["params"], report=rep)
    _say(f"  grads rel L2 {rep}")


def test_training_config_full_size_sampled():
    """300k primitives, SH degree 3 x order 2, 1352x1014, random time."""
    _say("[300k @ 1352x1014, sampled tiles]")
    _sampled_parity(scenegen.make_workload(1), 0, 10, seed=1, dl_seed=12)


def _sampled_forward(wl, views, n_tiles, seed):
    r, _ = PT.gpu_setup(wl.scene)
    rgb, dep, alp = r.render(wl.cameras, [float(x) for x in wl.times])
    items = r.split(rgb, dep, alp)
    stats = r.stats()
    _say(f"  active per view {stats['active_per_view']}, instances {stats['instances']}")
    for v in views:
        cam, t = wl.cameras[v], float(wl.times[v])
        tiles = scenegen.sample_pixels_dlddi(seed + v, [cam], n_tiles)[0].tolist()
        _, img = PT.oracle_view(wl.scene, cam, t, tiles=tiles)
        res = PT.compare_images(*(_np(x) for x in items[v]), img)
        _say(f"  view {v} ({cam.width}x{cam.height}) {res}")
    return r


def test_batched_forward_1m_16_mixed_views_sampled():
    """1M primitives with short lifetimes, 16 views at 800x800 and 1352x1014,
    one batched call; sampled tiles of one view of each size."""
    _say("[1M, 16 mixed views, sampled tiles]")
    _sampled_forward(scenegen.make_workload(2), [0, 1], 6, seed=20)


def test_batched_fwd_bwd_500k_8_views():
    """500k primitives, 8 views at 1352x1014, L2 loss: the batched gradient,
    taken through the torch.autograd wrapper, equals the sum of the per-view
    plain backwards, and sampled tiles of two views match the oracle in value
    and gradient."""
    _say("[500k, 8 views, fwd+bwd]")
    from paper_2310_10642_amd import g4d
    wl = scenegen.make_workload(3)
    r, params = PT.gpu_setup(wl.scene)
    times = [float(x) for x in wl.times]
    target = torch.from_numpy(np.concatenate([x.reshape(-1) for x in wl.targets])).cuda()
    scale = 1.0 / (3 * wl.cameras[0].width * wl.cameras[0].height)
    leaves = [p.clone().requires_grad_(True) for p in params]
    rgb = g4d.render(r, wl.cameras, times, *leaves)[0]
    (scale * ((rgb - target) ** 2).sum()).backward()      # L2, per-view mean, summed over views
    gb = [x.grad for x in leaves]
    dl = (2.0 * scale) * (rgb.detach() - target)
    gsum = r.grad_buffers()
    o = 0
    for v, (c, t) in enumerate(zip(wl.cameras, times)):
        n3 = 3 * c.width * c.height
        r.render([c], [t], depth=False, alpha=False)
        r.backward(dl[o:o + n3], out=gsum, accumulate=v > 0)
        o += n3
    torch.cuda.synchronize()
    for name, a, b in zip(PT.GROUPS, gb, gsum):
        a, b = _np(a).astype(np.float64), _np(b).astype(np.float64)
        nb = np.linalg.norm(b)
        assert nb == 0 or np.linalg.norm(a - b) <= 1e-5 * nb, name
    # oracle on sampled tiles of views 0 and 5
    sel = [0, 5]
    outs = []
    dls = []
    total = torch.zeros((), dtype=torch.float64)
    params_o = O.params_from_scene(wl.scene, requires_grad=True)
    for v in sel:
        cam, t = wl.cameras[v], times[v]
        tiles = scenegen.sample_pixels_dlddi(30 + v, [cam], 5)[0].tolist()
        out = O.render_view(params_o, cam, PT.f32(t), wl.scene.sh_degree, wl.scene.t_order, wl.scene.t_period,
                            tiles=tiles)
        img = dict(rgb=O.assemble(out, cam, "rgb", 3), depth=O.assemble(out, cam, "depth"),
                   alpha=O.assemble(out, cam, "alpha"), unc=O.assemble(out, cam, "uncertain"),
                   unc_g=O.assemble(out, cam, "uncertain_grad"))
        for c in PT.CAUSES:
            img["cause_" + c] = O.assemble(out, cam, "cause_" + c)
        rendered = ~np.isnan(img["depth"].detach().numpy())
        mask = (rendered & ~img["unc_g"].numpy()).astype(np.float64)
        drgb, _, _ = PT.dl_maps(40 + v, cam.height, cam.width, mask)
        total = total + O.tile_linear_loss(out, torch.as_tensor(drgb), cam=cam)
        outs.append((v, img))
        dls.append((v, drgb))
    total.backward()
    rgb, dep, alp = r.render(wl.cameras, times)
    items = r.split(rgb, dep, alp)
    for v, img in outs:
        res = PT.compare_images(*(_np(x) for x in items[v]), img)
        _say(f"  view {v} {res}")
    full = [np.zeros((3, c.height, c.width), np.float32) for c in wl.cameras]
    for v, d in dls:
        full[v] = d.astype(np.float32)
    g = r.backward(torch.from_numpy(np.concatenate([x.reshape(-1) for x in full])).cuda())
    torch.cuda.synchronize()
    rep = {}
    PT.compare_grads(g, params_o, report=rep)
    _say(f"  grads rel L2 {rep}")


def test_rounds_match_one_round():
    """Caps that split 8 views into rounds (including a round that is over the
    instance cap and binned again) change nothing per view: images and
    per-pixel state bit for bit, counters exactly, gradients up to the order
    of the sums. One view over the cap is a capacity error."""
    _say("[rounds vs one round, 300k x 8 views]")
    from paper_2310_10642_amd import g4d
    wl = scenegen.bench_workload(8)
    r, _ = PT.gpu_setup(wl.scene)
    times = [float(x) for x in wl.times]
    n = wl.scene.means4.shape[0]
    one = r.render(wl.cameras, times)
    s1 = r.stats()
    pt1, pl1 = r.debug("pix_t"), r.debug("pix_last")
    assert s1["rounds"] == 1
    assert s1["max_tile_list"] == int(np.diff(r.debug("ranges").reshape(-1, 2), axis=1).max())
    dl = torch.from_numpy(np.random.default_rng(55).uniform(-1, 1, one[0].numel()).astype(np.float32)).cuda()
    g1 = [x.clone() for x in r.backward(dl)]
    r.set_tuning(g4d.G4D_TUNE_ROUND_INSTANCES, s1["instances"] // 3)
    r.set_tuning(g4d.G4D_TUNE_ROUND_PAIRS, 3 * n)
    many = r.render(wl.cameras, times)
    s2 = r.stats()
    _say(f"  rounds {s2['rounds']}, instances {s1['instances']}")
    assert s2["rounds"] >= 3
    for a, b in zip(one, many):
        assert torch.equal(a, b)
    assert np.array_equal(pt1, r.debug("pix_t")) and np.array_equal(pl1, r.debug("pix_last"))
    for k in ("active_total", "instances", "fragments", "max_tile_list", "active_per_view", "tiles"):
        assert s1[k] == s2[k], k
    g2 = r.backward(dl)
    torch.cuda.synchronize()
    for name, a, b in zip(PT.GROUPS, g1, g2):
        a, b = _np(a).astype(np.float64), _np(b).astype(np.float64)
        nb = np.linalg.norm(b)
        assert nb == 0 or np.linalg.norm(a - b) <= 1e-5 * nb, name
    r.set_tuning(g4d.G4D_TUNE_ROUND_INSTANCES, 10)
    with pytest.raises(g4d.G4DError) as ei:
        r.render(wl.cameras[:1], times[:1])
    assert ei.value.status == g4d.G4D_ECAPACITY
    r.set_tuning(g4d.G4D_TUNE_ROUND_INSTANCES, 1 << 30)
    r.set_tuning(g4d.G4D_TUNE_ROUND_PAIRS, 1 << 28)
    again = r.render(wl.cameras, times)
    assert r.stats()["rounds"] == 1 and torch.equal(again[0], one[0])


def _close_grads(ga, gb, rel=1e-5):
    for name, a, b in zip(PT.GROUPS, ga, gb):
        a, b = _np(a).astype(np.float64), _np(b).astype(np.float64)
        assert np.isfinite(a).all(), name
        nb = np.linalg.norm(b)
        assert nb == 0 or np.linalg.norm(a - b) <= rel * nb, name


def test_sync_free_and_graph_replay():
    """The sync-free mode reproduces the synchronous training step (images bit
    for bit, loss and gradients up to summation order); a HIP graph captured
    around render + loss + backward replays it, three times, with eager work
    and synchronisation between the replays; the same with the loss folded
    into the backward."""
    _say("[sync-free and graph replay, 300k x 2 views]")
    from paper_2310_10642_amd import g4d
    wl = scenegen.bench_workload(2)
    r, _ = PT.gpu_setup(wl.scene)
    times = [float(x) for x in wl.times]
    tgt = torch.from_numpy(np.concatenate([x.reshape(-1) for x in wl.targets])).cuda()
    scale = 1.0 / (3 * wl.cameras[0].width * wl.cameras[0].height)

    def buffers():
        return (torch.empty_like(tgt), torch.empty(tgt.numel() // 3, device="cuda"),
                torch.empty(tgt.numel() // 3, device="cuda"), torch.zeros(1, device="cuda"), torch.empty_like(tgt))

    def step(grads, bufs):
        rgb, dep, alp, loss, dl = bufs
        r.render(wl.cameras, times, out=(rgb, dep, alp))
        loss.zero_()
        r.image_loss(g4d.G4D_LOSS_L1, rgb, tgt, scale, loss, dl)
        r.backward(dl, out=grads)
        return rgb, dep, alp, loss

    g_ref = r.grad_buffers()
    ref = step(g_ref, buffers())
    s_ref = r.stats()
    r.set_tuning(g4d.G4D_TUNE_SYNC_FREE, 1)
    g_sf = r.grad_buffers()
    sf = step(g_sf, buffers())
    s_sf = r.stats()
    for a, b in zip(ref[:3], sf[:3]):
        assert torch.equal(a, b)
    # the loss sums ~1e3 block partials with float atomics in any order
    loss_tol = 1e-5 * abs(float(ref[3]))
    assert abs(float(sf[3]) - float(ref[3])) <= loss_tol
    _close_grads(g_sf, g_ref)
    for k in ("active_total", "instances", "fragments", "max_tile_list", "active_per_view", "rounds"):
        assert s_ref[k] == s_sf[k], k

    g_gr = r.grad_buffers()
    bufs = buffers()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        outs = step(g_gr, bufs)
    for rep in range(3):
        for t in (*outs, *g_gr):
            t.fill_(float("nan"))
        x = torch.randn(512, 512, device="cuda")
        _ = float((x @ x).sum())               # eager work and a synchronisation
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(ref[:3], outs[:3]):
            assert torch.equal(a, b), rep
        assert abs(float(outs[3]) - float(ref[3])) <= loss_tol, rep
        _close_grads(g_gr, g_ref)
        _say(f"  replay {rep} ok")
    del graph

    # the same step with the loss folded into the backward, captured and
    # replayed: its loss sums have a fixed order, so every replay gives the
    # eager loss bit for bit
    def step_folded(grads, bufs):
        rgb, dep, alp, loss, _ = bufs
        r.render(wl.cameras, times, out=(rgb, dep, alp))
        loss.zero_()
        r.backward_loss(g4d.G4D_LOSS_L1, rgb, tgt, scale, loss, out=grads)
        return rgb, dep, alp, loss

    g_fe = r.grad_buffers()
    fe = step_folded(g_fe, buffers())
    torch.cuda.synchronize()
    assert abs(float(fe[3]) - float(ref[3])) <= loss_tol
    _close_grads(g_fe, g_ref)
    g_fg = r.grad_buffers()
    bufs = buffers()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        outs = step_folded(g_fg, bufs)
    for rep in range(3):
        for t in (*outs, *g_fg):
            t.fill_(float("nan"))
        x = torch.randn(512, 512, device="cuda")
        _ = float((x @ x).sum())
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(ref[:3], outs[:3]):
            assert torch.equal(a, b), rep
        assert torch.equal(outs[3], fe[3]), rep
        _close_grads(g_fg, g_ref)
        _say(f"  folded-loss replay {rep} ok")
    del graph
    r.set_tuning(g4d.G4D_TUNE_SYNC_FREE, 0)


@pytest.mark.parametrize("name,mk_scene,mk_cam,t,bg", CASES, ids=[c[0] for c in CASES])
def test_flow_parity(name, mk_scene, mk_cam, t, bg):
    """Rendered optical flow (two planes) against the oracle's, away from
    pixels with a decision FP32 may take the other way; the flow render keeps
    no state for a backward, and a render after it is unaffected."""
    _say(f"[flow parity] {name}")
    from paper_2310_10642_amd import g4d
    scene, cam = mk_scene(), mk_cam()
    dt = 0.05
    r, _ = PT.gpu_setup(scene, bg)
    t2 = t + 0.01                                  # a second view at another time
    flow = _np(r.render_flow([cam, cam], [t, t2], dt)).reshape(2, 2, cam.height, cam.width)
    with pytest.raises(g4d.G4DError):
        r.backward(torch.zeros(3 * cam.width * cam.height, device="cuda"))
    g_rgb, _, _ = _render_one(r, cam, t)
    _, img = PT.oracle_view(scene, cam, t, bg)
    assert np.abs(g_rgb - img["rgb"].numpy())[:, ~img["unc"].numpy()].max() <= PT.IMG_ATOL
    for v, tv in enumerate((t, t2)):
        out = O.render_flow(scene, cam, PT.f32(tv), PT.f32(dt))
        ref = O.assemble(out, cam, "rgb", 3)[:2].detach().numpy()
        # value flags: a decision FP32 may flip moves the blend weights by at
        # most 1e-5 at unflagged pixels, i.e. the flow by 1e-5 x a few pixels
        unc = O.assemble(out, cam, "uncertain").numpy()
        ok = ~unc
        err = np.abs(flow[v] - ref)[:, ok]
        tol = 1e-4 * (1.0 + np.abs(ref)[:, ok])
        _say(f"  view {v}: max |flow| {np.abs(ref).max():.3g} px, max err {err.max():.3g}, "
             f"flagged {unc.mean():.3%}")
        assert unc.sum() <= max(2, PT.MAX_FLAG_FRAC * unc.size) and (err <= tol).all()
        assert np.abs(ref).max() > 1e-3           # the scene moves


def test_densify_stats_parity():
    """Densification statistics of two views in one batch against the
    oracle's: per-view |dL/d(u,v)|, |dL/dmu_t| and the blended-view count.
    Counts agree exactly except at primitives whose blended-or-not decision
    in a view the oracle flags as within FP32 reach (they may differ by at
    most that many views); the sums agree where the counts do. The same batch
    split into two rounds accumulates the same values."""
    _say("[densification statistics, 3000 primitives x 2 views]")
    from paper_2310_10642_amd import g4d
    scene = _big_splat_scene(5, 3000, grow=0.8)
    cams = [scenegen.look_at_camera((1.0, 0.5, 3.5), 100, 70), scenegen.look_at_camera((-1.2, -0.2, 3.2), 96, 64)]
    times = [0.37, 0.52]
    dls = []
    for v, (cam, t) in enumerate(zip(cams, times)):
        _, img = PT.oracle_view(scene, cam, t)
        mask = (~img["unc_g"].numpy()).astype(np.float64)
        dls.append(PT.dl_maps(60 + v, cam.height, cam.width, mask)[0])
    uv_o, t_o, cnt_o, unsure = (x.numpy() for x in O.densify_stats(scene, cams, [PT.f32(x) for x in times], dls))
    r, _ = PT.gpu_setup(scene)
    n = scene.n
    dl = torch.from_numpy(np.concatenate([d.reshape(-1) for d in dls]).astype(np.float32)).cuda()
    runs = []
    for pairs in (1 << 28, n):                       # one round, then one view per round
        acc = (torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda"),
               torch.zeros(n, dtype=torch.int32, device="cuda"))
        r.set_tuning(g4d.G4D_TUNE_ROUND_PAIRS, pairs)
        r.set_densify_stats(*acc)
        r.render(cams, times)
        r.backward(dl)
        torch.cuda.synchronize()
        assert r.stats()["rounds"] == (1 if pairs > n else 2)
        runs.append([_np(x) for x in acc])
    uv_g, t_g, cnt_g = runs[0]
    diff = np.abs(cnt_g.astype(np.int64) - cnt_o)
    _say(f"  {int((cnt_o > 0).sum())} primitives blended somewhere; {int((unsure > 0).sum())} with a flagged "
         f"blend decision; counts differ at {int((diff > 0).sum())}")
    assert (cnt_o > 0).sum() > 100
    assert (diff <= unsure).all(), np.nonzero(diff > unsure)[0][:10]
    same = (diff == 0) & (unsure == 0)
    for name, a, b in (("uv", uv_g, uv_o), ("t", t_g, t_o)):
        a, b = a[same].astype(np.float64), b[same]
        assert np.linalg.norm(a - b) <= 1e-3 * np.linalg.norm(b), name
        rms = np.sqrt(np.mean(b * b))
        assert (np.abs(a - b) <= 1e-3 * (np.abs(b) + rms)).all(), name
    assert np.array_equal(runs[1][2], cnt_g)
    for a, b in zip(runs[1][:2], runs[0][:2]):
        assert np.allclose(a, b, rtol=1e-5, atol=1e-7 * float(np.abs(b).max()))
    r.set_densify_stats(None, None, None)


def test_tile_order_and_autotune():
    """Heavy-first tile order, the rasterisers' tile queue (resident or a
    given number of workgroups), the forward's LDS batch and the
    autotuner's choice among them change no result: images bit for bit,
    gradients up to the order of the atomic sums."""
    _say("[tile order and autotune, 300k x 2 views]")
    from paper_2310_10642_amd import g4d
    wl = scenegen.bench_workload(2)
    r, _ = PT.gpu_setup(wl.scene)
    times = [float(x) for x in wl.times]
    r.set_tuning(g4d.G4D_TUNE_TILE_ORDER, 0)
    ref = r.render(wl.cameras, times)
    dl = torch.from_numpy(np.random.default_rng(56).uniform(-1, 1, ref[0].numel()).astype(np.float32)).cuda()
    g_ref = [x.clone() for x in r.backward(dl)]
    with pytest.raises(g4d.G4DError):             # no heavy-first order to read
        r.debug("tile_order")
    r.set_tuning(g4d.G4D_TUNE_TILE_ORDER, 1)
    with pytest.raises(g4d.G4DError):             # the order change invalidated the kept state
        r.backward(dl)
    out = r.render(wl.cameras, times)
    for a, b in zip(ref, out):
        assert torch.equal(a, b)
    # the order: every tile once, by non-increasing list-length bin
    order, ranges = r.debug("tile_order").astype(np.int64), r.debug("ranges").astype(np.int64)
    assert np.array_equal(np.sort(order), np.arange(len(ranges)))
    lengths = (ranges[:, 1] - ranges[:, 0])[order].astype(np.float64)
    # bins of 2^(1/16) in len + 1, heaviest first; one bin of slack for the
    # device's fast log2 at a bin edge
    assert (lengths[1:] + 1 <= (lengths[:-1] + 1) * 2 ** (2 / 16)).all()
    # the longest list is the one the stats report, and the first tile is in its bin
    assert lengths.max() == r.stats()["max_tile_list"]
    assert lengths[0] + 1 >= (lengths.max() + 1) * 2 ** (-2 / 16)
    _close_grads(r.backward(dl), g_ref)
    for key, val in ((g4d.G4D_TUNE_PERSISTENT_BLOCKS, -1), (g4d.G4D_TUNE_PERSISTENT_BLOCKS, 37),
                     (g4d.G4D_TUNE_LDS_BATCH, 64), (g4d.G4D_TUNE_LDS_BATCH, 128)):
        r.set_tuning(key, val)
        assert r.get_tuning(key) == val
        out = r.render(wl.cameras, times)
        for a, b in zip(ref, out):
            assert torch.equal(a, b), (key, val)
        _close_grads(r.backward(dl), g_ref)
    r.set_tuning(g4d.G4D_TUNE_PERSISTENT_BLOCKS, 0)
    r.set_tuning(g4d.G4D_TUNE_LDS_BATCH, 256)
    with pytest.raises(g4d.G4DError):
        r.set_tuning(g4d.G4D_TUNE_LDS_BATCH, 100)
    r.set_tuning(g4d.G4D_TUNE_AUTOTUNE, 1)
    assert r.get_tuning(g4d.G4D_TUNE_AUTOTUNE) == 1
    out = r.render(wl.cameras, times)
    assert r.get_tuning(g4d.G4D_TUNE_AUTOTUNE) == 0
    blocks, order = r.get_tuning(g4d.G4D_TUNE_SORT_BLOCKS), r.get_tuning(g4d.G4D_TUNE_TILE_ORDER)
    pers, batch = r.get_tuning(g4d.G4D_TUNE_PERSISTENT_BLOCKS), r.get_tuning(g4d.G4D_TUNE_LDS_BATCH)
    _say(f"  autotune chose sort blocks {blocks}, tile order {order}, persistent {pers}, LDS batch {batch}")
    assert blocks in (512, 1024, 1280, 2048) and order in (0, 1) and pers in (0, -1) and batch in (64, 128, 256)
    for a, b in zip(ref, out):
        assert torch.equal(a, b)
    _close_grads(r.backward(dl), g_ref)


def _last_ids_batch(r, cams):
    """Per pixel of a one-round batch (views concatenated), view * n +
    primitive of the last contributor, -1 where none."""
    last = r.debug("pix_last").astype(np.int64)
    vals, ranges, ids = r.debug("tile_vals"), r.debug("ranges"), r.debug("ids").astype(np.int64)
    out, pix0, tile0 = [], 0, 0
    for cam in cams:
        tx, ty = (cam.width + 15) // 16, (cam.height + 15) // 16
        ys, xs = np.mgrid[0:cam.height, 0:cam.width]
        tile = tile0 + (ys // 16) * tx + (xs // 16)
        lv = last[pix0:pix0 + cam.width * cam.height].reshape(cam.height, cam.width)
        pos = np.clip(ranges[tile, 0].astype(np.int64) + lv - 1, 0, max(len(vals) - 1, 0))
        out.append(np.where(lv > 0, ids[vals[pos]] if len(vals) else -1, -1).ravel())
        pix0 += cam.width * cam.height
        tile0 += tx * ty
    return np.concatenate(out)


def test_ellipse_cull_is_exact():
    """Binning records only into the tiles their alpha-floor ellipse reaches
    and walking, per wave, only the entries whose ellipse meets its quadrant
    changes nothing against whole rectangles and every entry, on needle-like
    footprints in a batch of views: images, transmittance and last
    contributors (as primitives) bit for bit, and the same (record, tile)
    pairs blended.
    Gradients agree up to the order of the FP64 atomic sums of the tiles'
    shares (each tile's share is the same float32 value in both modes; the
    modes visit tiles in different orders): 1e-6 of the norm."""
    _say("[ellipse cull is exact]")
    from paper_2310_10642_amd import g4d
    scene = _needle_scene(12, 6000, 2.0, 1.5)
    cams = [scenegen.look_at_camera((math.sin(a) * 3.2, 0.25, math.cos(a) * 3.2), w, h)
            for a, (w, h) in zip([0.0, 1.7, 3.6], [(160, 120), (131, 97), (64, 200)])]
    times = [0.3, 0.55, 0.8]
    r, _ = PT.gpu_setup(scene, (0.1, 0.2, 0.3))
    dl = None
    got, inst = [], []
    for cull in (0, 1, 1):
        r.set_tuning(g4d.G4D_TUNE_ELLIPSE_CULL, cull)
        assert r.get_tuning(g4d.G4D_TUNE_ELLIPSE_CULL) == cull
        out = [x.clone() for x in r.render(cams, times)]
        inst.append(r.stats()["instances"])
        state = [r.debug("pix_t").copy(), _last_ids_batch(r, cams)]
        if dl is None:
            dl = torch.from_numpy(np.random.default_rng(4).uniform(-1, 1, out[0].numel()).astype(np.float32)).cuda()
        acc = (torch.zeros(scene.n, device="cuda"), torch.zeros(scene.n, device="cuda"),
               torch.zeros(scene.n, dtype=torch.int32, device="cuda"))
        r.set_densify_stats(*acc)
        g = [_np(x).astype(np.float64) for x in r.backward(dl)]
        r.set_densify_stats(None, None, None)
        got.append((out, state, g, _np(acc[2])))
    (o0, s0, g0, b0), (o1, s1, g1, b1), (_, _, g2, _) = got
    assert inst[1] < inst[0]
    for a, b in zip(o0, o1):
        assert torch.equal(a, b)
    for a, b in zip(s0, s1):
        assert np.array_equal(a, b)
    assert np.array_equal(b0, b1) and b0.sum() > 0
    for name, a, b, c in zip(PT.GROUPS, g0, g1, g2):
        nb = np.linalg.norm(b)
        spread = np.linalg.norm(c - b)
        _say(f"  {name}: |cull - all| / |g| = {np.linalg.norm(a - b) / max(nb, 1e-30):.2e}, "
             f"two runs {spread / max(nb, 1e-30):.2e}")
        assert np.isfinite(a).all() and np.linalg.norm(a - b) <= 1e-6 * nb, name


def test_sync_free_arena_overflow():
    """A sync-free render that needs more tile instances than the arena holds
    renders background only, its backward gives zero gradients, and get_stats
    reports the overflow once; a synchronous render then works."""
    _say("[sync-free arena overflow]")
    from paper_2310_10642_amd import g4d
    wl = scenegen.make_workload(0)
    cam = wl.cameras[0]
    r, _ = PT.gpu_setup(wl.scene)
    ref, _, _ = r.render([cam], [0.5])
    need = r.stats()["instances"]
    r2, _ = PT.gpu_setup(wl.scene)
    r2.render([cam], [50.0])                   # every primitive culled in time: a near-empty arena
    assert r2.stats()["instances"] == 0 < need
    r2.set_tuning(g4d.G4D_TUNE_SYNC_FREE, 1)
    rgb, _, alp = r2.render([cam], [0.5])
    g = r2.backward(torch.ones_like(rgb))
    torch.cuda.synchronize()
    assert float(rgb.abs().max()) == 0.0 and float(alp.abs().max()) == 0.0
    assert all(float(x.abs().max()) == 0.0 for x in g)
    with pytest.raises(g4d.G4DError) as ei:
        r2.stats()
    assert ei.value.status == g4d.G4D_ECAPACITY and str(need) in str(ei.value)
    assert r2.stats()["instances"] == 0       # reported once
    r2.set_tuning(g4d.G4D_TUNE_SYNC_FREE, 0)
    again, _, _ = r2.render([cam], [0.5])
    assert torch.equal(again, ref)
    r2.set_tuning(g4d.G4D_TUNE_SYNC_FREE, 1)
    again2, _, _ = r2.render([cam], [0.5])     # the arena now fits
    assert torch.equal(again2, ref) and r2.stats()["instances"] == need


@pytest.mark.timeout(400)
def test_long_sequence_3m_240_views_sampled():
    """3M short-lived primitives over 60 frames x 4 cameras at 1920x1080 in one
    call (several rounds under the default caps); sampled tiles of two views
    against the oracle."""
    _say("[3M, 240 views 1080p, sampled tiles]")
    wl = scenegen.make_workload(4)
    _say("  scene drawn")
    r = _sampled_forward(wl, [0, 237], 4, seed=70)
    s = r.stats()
    _say(f"  rounds {s['rounds']}, max list {s['max_tile_list']}, fragments {s['fragments']}")
    assert s["rounds"] >= 2 and s["n_views"] == 240


def test_image_loss_kernel():
    _say("[image loss]")
    from paper_2310_10642_amd import g4d
    r = g4d.Renderer(1, 1)
    rng = np.random.default_rng(9)
    n = 3 * 1000 + 7
    img, tgt = rng.uniform(size=n).astype(np.float32), rng.uniform(size=n).astype(np.float32)
    tgt[:5] = img[:5]                      # exact ties: zero L1 gradient
    I, Tg = torch.from_numpy(img).cuda(), torch.from_numpy(tgt).cuda()
    for kind, ref_l, ref_g in [(g4d.G4D_LOSS_L1, np.abs(img - tgt.astype(np.float64)).sum(),
                                np.sign(img.astype(np.float64) - tgt)),
                               (g4d.G4D_LOSS_L2, ((img.astype(np.float64) - tgt) ** 2).sum(),
                                2 * (img.astype(np.float64) - tgt))]:
        loss = torch.zeros(1, device="cuda")
        grad = torch.empty(n, device="cuda")
        r.image_loss(kind, I, Tg, 0.5, loss, grad)
        torch.cuda.synchronize()
        assert abs(float(loss) - 0.5 * ref_l) <= 1e-5 * 0.5 * ref_l
        assert np.allclose(_np(grad), 0.5 * ref_g, rtol=1e-6, atol=1e-7)


@pytest.mark.parametrize("n,off", [(1, 0), (2047, 0), (2052, 1), (524288, 0), (524293, 0), (2000003, 3)])
def test_image_loss_blocks(n, off):
    """The image loss around its 512-thread workgroups, one to 256 of them, on
    aligned and unaligned images. Every term is >= 0, so the sum is off by at most
    2^-24 of itself per addition of the longest chain: a thread's own, 6 in the
    wave, 8 over the waves, 256 workgroups, and 4 roundings of a term and its
    scale."""
    from paper_2310_10642_amd import g4d
    r = g4d.Renderer(1, 1)
    gen = torch.Generator().manual_seed(n)
    img, tgt = torch.rand(n + off, generator=gen)[off:], torch.rand(n + off, generator=gen)[off:]
    I, Tg = (torch.cat([torch.zeros(off), x]).cuda()[off:] for x in (img, tgt))
    d = img.double() - tgt.double()
    for kind, ref, rg in [(g4d.G4D_LOSS_L1, d.abs().sum(), d.sign()), (g4d.G4D_LOSS_L2, (d * d).sum(), 2 * d)]:
        loss = torch.zeros(1, device="cuda")
        grad = torch.empty(n + off, device="cuda")[off:]
        r.image_loss(kind, I, Tg, 0.5, loss, grad)
        bound = (-(-n // (512 * 256)) + 4 + 6 + 8 + 256 + 4) * 2.0**-24
        assert abs(float(loss) - 0.5 * float(ref)) <= bound * 0.5 * float(ref)
        assert torch.allclose(grad.cpu().double(), 0.5 * rg, rtol=2.0**-22, atol=0)


def test_backward_loss_equals_loss_then_backward():
    """The image loss folded into the backward (g4d_render_backward_loss) gives
    what g4d_image_loss followed by g4d_render_backward gives: gradients up to
    the order of the FP64 atomic sums, and the loss within float32 summation
    error of its FP64 value; over one round and over several rounds, L1 and
    L2, with and without a depth/alpha gradient."""
    _say("[backward with the loss folded in, 300k x 8 views]")
    from paper_2310_10642_amd import g4d
    wl = scenegen.bench_workload(8)
    r, _ = PT.gpu_setup(wl.scene)
    times = [float(x) for x in wl.times]
    n = wl.scene.means4.shape[0]
    target_np = np.concatenate([t.reshape(-1) for t in wl.targets]).astype(np.float32)
    target = torch.from_numpy(target_np).cuda()
    scale = 1.0 / target.numel()
    rng = np.random.default_rng(12)
    for rounds, kind, with_alpha in [(False, g4d.G4D_LOSS_L1, False), (False, g4d.G4D_LOSS_L2, True),
                                     (True, g4d.G4D_LOSS_L1, False)]:
        if rounds:
            r.set_tuning(g4d.G4D_TUNE_ROUND_PAIRS, 3 * n)
        rgb, _, alpha = r.render(wl.cameras, times)
        assert (r.stats()["rounds"] >= 3) == rounds
        dla = (torch.from_numpy(rng.uniform(-1, 1, alpha.numel()).astype(np.float32)).cuda()
               if with_alpha else None)
        loss_a = torch.zeros(1, device="cuda")
        dl = torch.empty_like(rgb)
        r.image_loss(kind, rgb, target, scale, loss_a, dl)
        ga = [x.clone() for x in r.backward(dl, None, dla)]
        loss_b = torch.zeros(1, device="cuda")
        gb = r.backward_loss(kind, rgb, target, scale, loss_b, None, dla)
        torch.cuda.synchronize()
        _close_grads(gb, ga, rel=1e-6)
        d = _np(rgb).astype(np.float64) - target_np
        ref = scale * (np.abs(d).sum() if kind == g4d.G4D_LOSS_L1 else (d * d).sum())
        _say(f"  rounds {r.stats()['rounds']} kind {kind}: loss {float(loss_b):.7g} "
             f"(image_loss {float(loss_a):.7g}, FP64 {ref:.7g})")
        for lv in (float(loss_a), float(loss_b)):
            assert abs(lv - ref) <= 1e-5 * ref
    r.set_tuning(g4d.G4D_TUNE_ROUND_PAIRS, 1 << 28)
    with pytest.raises(g4d.G4DError) as ei:
        r.backward_loss(7, rgb, target, scale, loss_b)
    assert ei.value.status == g4d.G4D_EINVAL


def test_stage_timing_and_stats():
    _say("[stage timing]")
    sc = _big_splat_scene(8, 2000)
    cam = scenegen.look_at_camera((0.0, 0.0, 3.5), 64, 64)
    r, _ = PT.gpu_setup(sc)
    r.stage_timing(True)
    r.render([cam, cam], [0.4, 0.6])
    r.backward(torch.ones(2 * 3 * 64 * 64, device="cuda"))
    st = r.stage_times()
    r.stage_timing(False)
    assert st["preprocess"][1] == 1 and st["binning"][1] == 2 and st["raster_fwd"][1] == 1
    # the preprocess backward's stage also times the zeroing of the gradient
    # lines; the colour pass is timed on its own stream
    assert st["raster_bwd"][1] == 1 and st["preprocess_bwd"][1] == 2 and st["colour"][1] == 1
    assert all(ms >= 0 for ms, _ in st.values())
    s = r.stats()
    assert s["n_views"] == 2 and sum(s["active_per_view"]) == s["active_total"] > 0
    last = r.debug("pix_last").astype(np.int64)
    assert s["fragments"] == int(last.sum())


def test_adam_step_matches_oracle():
    """Three fused Adam steps over all six groups against the FP64 oracle."""
    _say("[adam step]")
    from oracle import optim as OP
    sc = scenegen.random_scene(35, 3000, sh_degree=3, t_order=2)
    r, params = PT.gpu_setup(sc)
    n, K = sc.n, sc.coeffs.shape[1]
    rng = np.random.default_rng(36)
    shapes = dict(means4=(n, 4), log_scales4=(n, 4), q_left=(n, 4), q_right=(n, 4), opacity_logit=(n,),
                  coeffs=(n, K, 3))
    lr = [1.6e-4, 5e-3, 1e-3, 1e-3, 5e-2, 2.5e-3]
    p_o = {g: getattr(sc, g).astype(np.float64) for g in OP.GROUPS}
    m_o = {g: np.zeros(shapes[g]) for g in OP.GROUPS}
    v_o = {g: np.zeros(shapes[g]) for g in OP.GROUPS}
    m = torch.zeros(n * (17 + 3 * K), device="cuda")
    v = torch.zeros_like(m)
    for step in (1, 2, 3):
        grads = {g: rng.normal(size=shapes[g]).astype(np.float32) for g in OP.GROUPS}
        r.adam_step(params, [torch.from_numpy(grads[g]).cuda() for g in OP.GROUPS], m, v, step, lr, eps=1e-8)
        # the oracle takes the float32 values the library receives
        f32 = lambda x: float(np.float32(x))
        p_o, m_o, v_o = OP.adam_step(p_o, grads, m_o, v_o, step, [f32(x) for x in lr], f32(0.9), f32(0.999),
                                     f32(1e-8))
    torch.cuda.synchronize()
    # FP32 forms each update lr (m / bc1) / (sqrt(v / bc2) + eps) to ~1e-6 of
    # its size (|u| <~ 3 over the first steps): three steps move p by at most
    # ~1e-5 lr beyond the rounding of p itself
    for gi, (g, t) in enumerate(zip(OP.GROUPS, params)):
        assert np.allclose(_np(t), p_o[g], rtol=2e-6, atol=1e-5 * lr[gi]), g
    off = 0
    for g in OP.GROUPS:
        cnt = int(np.prod(shapes[g]))
        assert np.allclose(_np(m)[off:off + cnt], m_o[g].reshape(-1), rtol=1e-5, atol=1e-7), g
        assert np.allclose(_np(v)[off:off + cnt], v_o[g].reshape(-1), rtol=1e-5, atol=1e-9), g
        off += cnt


def test_split_sample_matches_oracle():
    """mu + R S z for random primitives and draws; an index outside [0, n)
    gives a NaN row and reads nothing."""
    _say("[split sample]")
    from oracle import optim as OP
    sc = scenegen.random_scene(37, 500)
    r, _ = PT.gpu_setup(sc)
    rng = np.random.default_rng(38)
    idx = rng.integers(0, sc.n, 2000).astype(np.int32)
    idx[7] = sc.n                                   # not a primitive
    z = rng.normal(size=(2000, 4)).astype(np.float32)
    out = _np(r.split_sample(torch.from_numpy(idx).cuda(), torch.from_numpy(z).cuda()))
    ok = np.arange(2000) != 7
    ref = OP.split_sample(sc, idx[ok], z[ok])
    assert np.isnan(out[7]).all()
    assert np.allclose(out[ok], ref, rtol=1e-5, atol=1e-6)


def _oracle_views_grad(scene, cams, times, tiles_per_view, dl_seed, bg=(0.0, 0.0, 0.0), planes=("rgb",)):
    """The oracle over sampled tiles of several views sharing one set of
    parameters: images per view, and the gradient of sum_v <dL/dI_v, I_v> for
    random output gradients (zero on gradient-flagged pixels) of the given
    planes. Returns (params, [(img, dl dict)] per view)."""
    params = O.params_from_scene(scene, requires_grad=True)
    total = torch.zeros((), dtype=torch.float64)
    views = []
    for v, (cam, t) in enumerate(zip(cams, times)):
        tiles = tiles_per_view[v]
        out = O.render_view(params, cam, PT.f32(t), scene.sh_degree, scene.t_order, scene.t_period, bg, tiles=tiles)
        img = dict(rgb=O.assemble(out, cam, "rgb", 3), depth=O.assemble(out, cam, "depth"),
                   alpha=O.assemble(out, cam, "alpha"), unc=O.assemble(out, cam, "uncertain"),
                   unc_g=O.assemble(out, cam, "uncertain_grad"))
        for c in PT.CAUSES:
            img["cause_" + c] = O.assemble(out, cam, "cause_" + c)
        rendered = ~np.isnan(img["depth"].detach().numpy())
        mask = (rendered & ~img["unc_g"].numpy()).astype(np.float64)
        drgb, ddep, dalp = PT.dl_maps(dl_seed + v, cam.height, cam.width, mask)
        dl = dict(rgb=drgb, depth=ddep if "depth" in planes else None, alpha=dalp if "alpha" in planes else None)
        total = total + O.tile_linear_loss(out, torch.as_tensor(drgb),
                                           None if dl["depth"] is None else torch.as_tensor(ddep),
                                           None if dl["alpha"] is None else torch.as_tensor(dalp), cam)
        views.append((img, dl))
    total.backward()
    return params, views


def _cat_planes(cams, per_view, key, channels):
    """Concatenated device buffer of one output-gradient plane (zeros where a
    view has none); None when no view has it."""
    if all(dl[key] is None for _, dl in per_view):
        return None
    parts = []
    for cam, (_, dl) in zip(cams, per_view):
        x = dl[key]
        parts.append(np.zeros((channels, cam.height, cam.width)) if x is None else x)
    return torch.from_numpy(np.concatenate([p.reshape(-1) for p in parts]).astype(np.float32)).cuda()


def test_bench_step_variants_match_oracle():
    """Exactly what the benchmark times: the 300k scene over 8 views at
    1352x1014 rendered with no depth or alpha planes, and the rgb-only
    backward; on sampled tiles of two views, the images and the gradients
    match the oracle. The backward with a depth plane only and with an alpha
    plane only (the other two compiled variants) match it too."""
    _say("[bench step variants, 300k x 8 views]")
    wl = scenegen.bench_workload(8)
    cams, times = wl.cameras, [float(x) for x in wl.times]
    sel = [2, 6]
    tiles = {v: scenegen.sample_pixels_dlddi(80 + v, [cams[v]], 4)[0].tolist() for v in sel}
    r, _ = PT.gpu_setup(wl.scene)
    rgb, dep, alp = r.render(cams, times, depth=False, alpha=False)
    assert dep is None and alp is None
    items = r.split(rgb)
    for planes in (("rgb",), ("rgb", "depth"), ("rgb", "alpha")):
        params, views = _oracle_views_grad(wl.scene, [cams[v] for v in sel], [times[v] for v in sel],
                                           [tiles[v] for v in sel], 90, planes=planes)
        if planes == ("rgb",):
            for v, (img, _) in zip(sel, views):
                g_rgb = _np(items[v][0])
                rendered = ~np.isnan(img["depth"].detach().numpy())
                ok = rendered & ~img["unc"].numpy()
                err = np.abs(g_rgb - img["rgb"].detach().numpy()).max(0)
                _say(f"  view {v}: max rgb err {float(err[ok].max()):.3g}, flags {PT.flag_report(img, rendered)}")
                assert (err[ok] <= PT.IMG_ATOL).all()
                assert (rendered & img["unc"].numpy()).sum() <= max(2, PT.MAX_FLAG_FRAC * rendered.sum())
        per_view = []
        for v, cam in enumerate(cams):
            per_view.append(views[sel.index(v)] if v in sel else (None, dict(rgb=None, depth=None, alpha=None)))
        dl_rgb = _cat_planes(cams, per_view, "rgb", 3)
        dl_dep = _cat_planes(cams, per_view, "depth", 1)
        dl_alp = _cat_planes(cams, per_view, "alpha", 1)
        if planes != ("rgb",):
            # the depth / alpha variants need a render that kept those planes' state
            r.render(cams, times, depth="depth" in planes, alpha="alpha" in planes)
        g = r.backward(dl_rgb, dl_dep, dl_alp)
        torch.cuda.synchronize()
        rep = {}
        PT.compare_grads(g, params, report=rep)
        _say(f"  backward {planes}: rel L2 {rep}")


def test_needle_scene_gradients_match_oracle_in_both_cull_modes():
    """The 6000-needle, 3-view scene of the ellipse-cull test: with the
    ellipse tests on and off, the batched gradients match the oracle's on
    sampled tiles of every view at the gradient tolerance (the needles add
    terms of both signs from many tiles in an order the two modes do not
    share)."""
    _say("[needles x 3 views: gradients in both cull modes]")
    from paper_2310_10642_amd import g4d
    scene = _needle_scene(12, 6000, 2.0, 1.5)
    cams = [scenegen.look_at_camera((math.sin(a) * 3.2, 0.25, math.cos(a) * 3.2), w, h)
            for a, (w, h) in zip([0.0, 1.7, 3.6], [(160, 120), (131, 97), (64, 200)])]
    times = [0.3, 0.55, 0.8]
    bg = (0.1, 0.2, 0.3)
    tiles = [scenegen.sample_pixels_dlddi(100 + v, [c], 10)[0].tolist() for v, c in enumerate(cams)]
    params, views = _oracle_views_grad(scene, cams, times, tiles, 110, bg=bg, planes=("rgb", "depth", "alpha"))
    r, _ = PT.gpu_setup(scene, bg)
    for cull in (1, 0):
        r.set_tuning(g4d.G4D_TUNE_ELLIPSE_CULL, cull)
        rgb, dep, alp = r.render(cams, times)
        for v, (img, _) in enumerate(views):
            # aspect ratios of ~33: the quadratic form of a fragment cancels
            # terms far larger than itself, which widens the float32 reach of
            # its alpha (Margins.alpha_fp32) and the flags with it
            res = PT.compare_images(*(_np(x) for x in r.split(rgb, dep, alp)[v]), img, max_flag_frac=1e-2)
            _say(f"  cull {cull} view {v}: {res}")
        g = r.backward(_cat_planes(cams, views, "rgb", 3), _cat_planes(cams, views, "depth", 1),
                       _cat_planes(cams, views, "alpha", 1))
        torch.cuda.synchronize()
        rep = {}
        PT.compare_grads(g, params, report=rep)
        _say(f"  cull {cull}: grads rel L2 {rep}")
    r.set_tuning(g4d.G4D_TUNE_ELLIPSE_CULL, 1)


def test_nonfinite_parameters_are_culled_and_counted():
    """Primitives with a NaN or infinite parameter are left out: one with a
    non-finite mean, scale, quaternion or opacity in every view, one with a
    non-finite 4DSH coefficient where it would otherwise be drawn (rendered
    fully transparent). Images equal, bit for bit, those of the scene without
    those primitives; stats count the pairs left out; their gradients are
    zero and every other gradient matches the scene without them."""
    _say("[non-finite parameters]")
    base = _big_splat_scene(5, 3000, grow=0.8)
    cams = [scenegen.look_at_camera((1.0, 0.5, 3.5), 100, 70), scenegen.look_at_camera((-1.2, -0.2, 3.2), 96, 64)]
    times = [0.37, 0.52]
    r, _ = PT.gpu_setup(base)
    r.render(cams, times)
    n = base.n
    ids = r.debug("ids").astype(np.int64)
    pairs = np.bincount(ids % n, minlength=n)              # active views per primitive
    visible = np.nonzero(pairs > 0)[0]
    rng = np.random.default_rng(7)
    pick = rng.choice(visible, size=12, replace=False)
    geo_bad, coef_bad = pick[:7], pick[7:]
    bad = scenegen.Scene(*(np.array(getattr(base, k)) for k in ("means4", "log_scales4", "q_left", "q_right",
                                                                "opacity_logit", "coeffs")),
                         base.sh_degree, base.t_order, base.t_period)
    nan, inf = np.float32(np.nan), np.float32(np.inf)
    bad.means4[geo_bad[0], 0] = nan
    bad.means4[geo_bad[1], 3] = -inf
    bad.log_scales4[geo_bad[2], 2] = inf
    bad.q_left[geo_bad[3], 1] = nan
    bad.q_right[geo_bad[4], 0] = -inf
    bad.opacity_logit[geo_bad[5]] = nan
    bad.log_scales4[geo_bad[6], 3] = nan
    bad.coeffs[coef_bad[0], 0, 0] = nan
    bad.coeffs[coef_bad[1], 3, 2] = inf
    bad.coeffs[coef_bad[2], 5, 1] = -inf
    bad.coeffs[coef_bad[3], 1, 0] = nan
    bad.coeffs[coef_bad[4], 2, 2] = inf
    keep = np.setdiff1d(np.arange(n), pick)
    clean = scenegen.Scene(base.means4[keep], base.log_scales4[keep], base.q_left[keep], base.q_right[keep],
                           base.opacity_logit[keep], base.coeffs[keep], base.sh_degree, base.t_order, base.t_period)
    rb, _ = PT.gpu_setup(bad)
    rc, _ = PT.gpu_setup(clean)
    out_b = [x.clone() for x in rb.render(cams, times)]
    st = rb.stats()
    out_c = [x.clone() for x in rc.render(cams, times)]
    for a, b in zip(out_b, out_c):
        assert torch.equal(a, b)
    want = len(geo_bad) * len(cams) + int(pairs[coef_bad].sum())
    _say(f"  culled_nonfinite {st['culled_nonfinite']} (expected {want})")
    assert st["culled_nonfinite"] == want
    assert rc.stats()["culled_nonfinite"] == 0
    dl = torch.from_numpy(np.random.default_rng(8).uniform(-1, 1, out_b[0].numel()).astype(np.float32)).cuda()
    gb = [_np(x).astype(np.float64) for x in rb.backward(dl)]
    gc = [_np(x).astype(np.float64) for x in rc.backward(dl)]
    for name, a, b in zip(PT.GROUPS, gb, gc):
        assert np.isfinite(a).all(), name
        assert (a[pick] == 0).all(), name
        nb = np.linalg.norm(b)
        assert np.linalg.norm(a[keep] - b) <= 1e-5 * nb, name


@pytest.mark.parametrize("views", [683, 1366, 3414])
def test_forward_quadrants_per_wave(views):
    """The forward rasteriser gives a wave one, two or four quadrants by the
    launch's tile count (12 tiles a view here, ragged at both edges: 8196 tiles, then
    16392 and 40968, just past its two lines). Every view equals its own small
    render bit for bit, with and without the depth plane, all in one launch
    and taken from the tile queue."""
    from paper_2310_10642_amd import g4d
    r, _ = PT.gpu_setup(_big_splat_scene(61, 400, grow=0.6, sh=1, to=1))
    cams = [scenegen.ring_camera(0.01 * v, 61, 45) for v in range(views)]
    times = [(v % 97) / 97.0 for v in range(views)]
    hw = 61 * 45
    for queue in (0, -1):
        r.set_tuning(g4d.G4D_TUNE_PERSISTENT_BLOCKS, queue)
        rgb, dep, alp = r.render(cams, times)
        flat = r.render(cams, times, depth=False, alpha=False)[0]
        assert torch.equal(flat, rgb)
        r.set_tuning(g4d.G4D_TUNE_PERSISTENT_BLOCKS, 0)
        for v in (0, 1, views // 2, views - 1):
            one = r.render([cams[v]], [times[v]])
            for got, want, k in zip((rgb, dep, alp), one, (3, 1, 1)):
                assert torch.equal(got[k * hw * v:k * hw * (v + 1)], want), (queue, v, k)


@pytest.mark.parametrize("views", [1710, 180])
@pytest.mark.parametrize("planes", ["rgb", "depth", "alpha", "both", "loss", "nan"])
def test_backward_one_wave_per_tile(planes, views):
    """A launch of 20480 or more tiles takes the one-wave-per-tile backward;
    the same views in two halves take the four-wave one. Below 2048 tiles the
    waves take two roles: 2160 tiles against twice 1080. Needle footprints
    (the FP64 moments) and opaque ones (the alpha clamp), ragged 61x45 images
    (12 tiles a view), odd counts of list entries.

    Both add the same terms: a tile's sums have 256 float32 terms, some 25
    roundings deep (1.5e-6 of the sum of their magnitudes), in another order,
    and their totals are added in FP64; 20 times that allows for the
    cancellation between terms of both signs. A non-finite output gradient
    makes the same values non-finite."""
    from paper_2310_10642_amd import g4d
    sc = _needle_scene(62, 151, 1.2, 0.8)
    sc.opacity_logit[::3] += np.float32(8.0)
    r, _ = PT.gpu_setup(sc)
    cams = [scenegen.ring_camera(0.01 * v, 61, 45) for v in range(views)]
    times = [(v % 97) / 97.0 for v in range(views)]
    hw, rng = 61 * 45, np.random.default_rng(63)
    dl = [torch.from_numpy(rng.uniform(-1, 1, k * hw * views).astype(np.float32)).cuda() for k in (3, 1, 1)]
    if planes == "nan":
        dl[0][5 * 3 * hw + hw + 777] = float("nan")
        dl[0][(views // 2 + 45) * 3 * hw + 1234] = float("inf")
    use = (planes in ("depth", "both"), planes in ("alpha", "both"))

    def run(v0, v1, grads, accumulate):
        rgb = r.render(cams[v0:v1], times[v0:v1])[0]
        a = [x[k * hw * v0:k * hw * v1].contiguous() for x, k in zip(dl, (3, 1, 1))]
        if planes == "loss":
            return r.backward_loss(g4d.G4D_LOSS_L2, rgb, a[0], 0.5, loss, out=grads, accumulate=accumulate)
        return r.backward(a[0], a[1] if use[0] else None, a[2] if use[1] else None, out=grads, accumulate=accumulate)

    loss = torch.zeros(1, device="cuda")
    g = [x.double().cpu() for x in run(0, views, None, False)]
    loss_one, loss = float(loss), torch.zeros(1, device="cuda")
    parts = run(0, views // 2, None, False)
    ref = [x.double().cpu() for x in run(views // 2, views, parts, True)]
    for a, b in zip(g, ref):
        fine = torch.isfinite(b)
        assert torch.equal(fine, torch.isfinite(a)) and (planes == "nan") == (not bool(fine.all()))
        a, b = torch.where(fine, a, 0.0), torch.where(fine, b, 0.0)
        assert float((a - b).norm()) <= 3e-5 * float(b.norm())
    assert planes != "loss" or abs(loss_one - float(loss)) <= 1e-5 * float(loss)


@pytest.mark.parametrize("n,views", [(1, 3), (63, 17), (257, 33), (65700, 64)])
def test_pair_listing_and_places(n, views):
    """Pairs are listed by units of 64 primitives and 16 views at a time, pass a
    single-precision bound of the temporal filter, and are compacted by
    256-pair groups (in two levels beyond 16384 of them: 257 a view in the last
    case). Every view equals its own render bit for bit, so no pair is lost,
    doubled or out of order; quaternions scaled by powers of two, whose squares
    leave single precision, change no bit either."""
    # short-lived primitives: most pairs are filtered
    sc = _big_splat_scene(67, n, grow=0.0 if n > 1000 else 0.4, sh=1, to=1, mu_log_t=-3.5)
    r, _ = PT.gpu_setup(sc)
    cams = [scenegen.ring_camera(0.07 * v, 45, 37) for v in range(views)]
    times = [(v * 7 % 31) / 31.0 for v in range(views)]
    rgb, dep, alp = r.render(cams, times)
    act = r.stats()["active_per_view"]
    hw = 45 * 37
    for v in range(views) if n < 1000 else (0, 1, 15, 16, 31, 62, 63):
        one = r.render([cams[v]], [times[v]])
        for got, want, k in zip((rgb, dep, alp), one, (3, 1, 1)):
            assert torch.equal(got[k * hw * v:k * hw * (v + 1)], want), (v, k)
        assert r.stats()["active_per_view"] == [act[v]]
    sc.q_left[::2] *= np.float32(2.0**66)
    sc.q_right[::3] *= np.float32(2.0**-66)
    assert torch.equal(PT.gpu_setup(sc)[0].render(cams, times)[0], rgb)


@pytest.mark.parametrize("n", [3300, 3601])
def test_large_tile_sort(n):
    """From 2^24 instances on the tile sort takes wider workgroups: six views of
    some 3M instances each (primitives that cover the whole image) equal the
    same views in rounds below the line, bit for bit."""
    from paper_2310_10642_amd import g4d
    r, _ = PT.gpu_setup(_big_splat_scene(71, n, grow=3.0, sh=1, to=1, mu_log_t=1.0))
    cams = [scenegen.ring_camera(0.3 * v, 512, 512) for v in range(6)]
    times = [0.1 * v for v in range(6)]
    one = r.render(cams, times)
    st = r.stats()
    assert st["rounds"] == 1 and st["instances"] >= 1 << 24
    r.set_tuning(g4d.G4D_TUNE_ROUND_INSTANCES, 1 << 23)
    many = r.render(cams, times)
    assert r.stats()["rounds"] in (3, 6)
    for a, b in zip(one, many):
        assert torch.equal(a, b)


@pytest.mark.parametrize("n,views", [(1, 1), (1024, 1), (1025, 1), (2048, 1), (2049, 1), (4097, 1), (8192, 1),
                                     (8193, 1), (2731, 3), (9000, 5), (40960, 8), (130000, 8)])
def test_small_sorts(n, views):
    """The sorts of few pairs: with the gather up to 2048, one workgroup of 4 or 8
    pairs a thread up to 8192, chained one-launch passes beyond, the three-launch
    passes past 3 * 2^18. Pairs at the depth of others (copies of primitives) keep
    their order: the records are in order of (depth, view, primitive), every tile's
    list in order of the records, on the first render and on the next (whose grid
    is another)."""
    sc = _big_splat_scene(73, n, grow=0.3 if n < 10000 else -1.5, sh=1, to=1, mu_log_t=1.0)
    sc.means4[n // 2:2 * (n // 2)] = sc.means4[:n // 2]
    r, _ = PT.gpu_setup(sc)
    cams = [scenegen.ring_camera(0.4 * v, 125, 77) for v in range(views)]
    for _ in range(2):
        r.render(cams, [0.5] * views)
        z, ids = r.debug("records")[:, 2], r.debug("ids").astype(np.int64)
        assert len(ids) == r.stats()["active_total"] and len(np.unique(ids)) == len(ids)
        if len(ids) > 1:
            dz, di = np.diff(z), np.diff(ids)
            assert (dz >= 0).all() and (di[dz == 0] > 0).all()
        vals, ranges = r.debug("tile_vals").astype(np.int64), r.debug("ranges").astype(np.int64)
        assert (ranges[:, 1] - ranges[:, 0]).sum() == len(vals) == r.stats()["instances"]
        step = np.diff(vals) > 0
        step[ranges[ranges[:, 0] < ranges[:, 1], 1][:-1] - 1] = True  # from one list to the next
        assert step.all()
        order = r.debug("tile_order").astype(np.int64)
        assert (np.sort(order) == np.arange(len(ranges))).all()


def test_counts_beyond_the_guess():
    """A render enqueues its binning and rasteriser for a guess at the counts from
    earlier renders. After renders of a far camera a near one exceeds the guess
    by far, then the other way round, and a round cap set in between cuts the
    call into rounds: images, statistics and tile lists are those of a new
    context, gradients up to the order of the atomic sums."""
    from paper_2310_10642_amd import g4d
    sc = _big_splat_scene(79, 6000, grow=0.2, sh=1, to=1, mu_log_t=0.5)
    far = [scenegen.look_at_camera((0.0, 0.3 * v, 40.0), 160, 120) for v in range(3)]
    near = [scenegen.look_at_camera((0.1 * v, 0.0, 2.6), 160, 120) for v in range(3)]
    r, _ = PT.gpu_setup(sc)
    times = [0.3, 0.5, 0.7]
    dl = torch.from_numpy(np.random.default_rng(80).uniform(-1, 1, 3 * 3 * 160 * 120).astype(np.float32)).cuda()
    for step, cams in enumerate((far, far, near, far, near[:1], near, near, far)):
        t = times[:len(cams)]
        if step == 5:
            r.set_tuning(g4d.G4D_TUNE_ROUND_INSTANCES, 2 * near_total // 3)
        f, _ = PT.gpu_setup(sc)
        got, want = r.render(cams, t), f.render(cams, t)
        for a, b in zip(got, want):
            assert torch.equal(a, b), step
        sg, sw = r.stats(), f.stats()
        if step == 2:
            near_total = sg["instances"]
        assert sg["rounds"] >= (2 if step in (5, 6) else 1)
        assert {**sg, "rounds": 0} == {**sw, "rounds": 0}, step
        if sg["rounds"] == 1:
            assert np.array_equal(r.debug("tile_vals"), f.debug("tile_vals"))
        d = dl[:got[0].numel()]
        _close_grads(r.backward(d), f.backward(d))


@pytest.mark.parametrize("every", [9, 40])
def test_emission_of_many_records(every):
    """From 2^20 records on the emission takes 128 of them a block, and a block's
    tile rows 1024 at a time: tall images (126 rows of tiles) with every 9th or
    40th primitive across the whole height, so that most blocks or few have
    more. Views of the one call equal their own renders (64 records a block)
    bit for bit, and the tile lists are in order."""
    sc = _big_splat_scene(83, 74000, grow=-2.5, sh=1, to=1, mu_log_t=1.0)
    sc.log_scales4[::every, :3] += np.float32(3.0)
    r, _ = PT.gpu_setup(sc)
    cams = [scenegen.ring_camera(0.1 * v, 40, 2010) for v in range(16)]
    times = [0.5] * 16
    rgb = r.render(cams, times, depth=False, alpha=False)[0]
    assert r.stats()["active_total"] >= 1 << 20 and r.stats()["rounds"] == 1
    vals, ranges = r.debug("tile_vals").astype(np.int64), r.debug("ranges").astype(np.int64)
    step = np.diff(vals) > 0
    step[ranges[ranges[:, 0] < ranges[:, 1], 1][:-1] - 1] = True
    assert step.all() and (ranges[:, 1] - ranges[:, 0]).sum() == len(vals)
    k = 3 * 40 * 2010
    for v in (0, 7, 15):
        assert torch.equal(rgb[k * v:k * (v + 1)], r.render([cams[v]], [0.5], depth=False, alpha=False)[0]), v



def _near_and_far_scene(seed, n_big, n_small):
    """n_big large primitives alive around t = 0.1 only, n_small tiny ones around 0.9."""
    sc = scenegen.random_scene(seed, n_big + n_small, sh_degree=1, t_order=1)
    sc.q_left[:], sc.q_right[:] = np.float32([1, 0, 0, 0]), np.float32([1, 0, 0, 0])
    sc.log_scales4[:, 3] = np.float32(-4.0)
    sc.log_scales4[:n_big, :3], sc.log_scales4[n_big:, :3] = np.float32(0.0), np.float32(-6.0)
    sc.opacity_logit[:] = np.float32(1.0)
    sc.means4[:, :3] *= np.float32(0.5)
    sc.means4[:n_big, 3], sc.means4[n_big:, 3] = np.float32(0.1), np.float32(0.9)
    return sc


@pytest.mark.parametrize("w,h,views,n_big", [(160, 120, 1, 1000), (160, 120, 3, 1000), (160, 120, 1, 200),
                                             (16, 16, 1, 1000)])
def test_records_beyond_the_guess(w, h, views, n_big):
    """A render whose records (and in two cases its instances) exceed the guess
    from earlier renders: few active primitives that cover the image, then
    20,000 active ones of a few tiles at most, and back. The stages enqueued
    for the guess may see no instance (they would read slots that nothing
    wrote): images, statistics (the longest list among them), tile lists and
    gradients are those of a new context. A 16x16 image has one tile, whose list takes no
    sort."""
    sc = _near_and_far_scene(91, n_big, 20000)
    r, _ = PT.gpu_setup(sc)
    cams = [scenegen.look_at_camera((0.2 * v, 0.1, 4.0), w, h) for v in range(views)]
    dl = torch.from_numpy(np.random.default_rng(92).uniform(-1, 1, 3 * w * h * views).astype(np.float32)).cuda()
    if w == 16:  # (an arena of more slots than the first single tile fills)
        r.render([scenegen.look_at_camera((0.0, 0.1, 4.0), 160, 120)], [0.1])
    most = 0  # active in one view so far
    for t in (0.1, 0.1, 0.9, 0.1, 0.9):
        f, _ = PT.gpu_setup(sc)
        got, want = r.render(cams, [t] * views), f.render(cams, [t] * views)
        for a, b in zip(got, want):
            assert torch.equal(a, b), t
        sg = r.stats()
        assert sg == f.stats(), t
        assert sg["max_tile_list"] == int(np.diff(r.debug("ranges").astype(np.int64), axis=1).max())
        if t == 0.9 and most <= n_big:
            assert sg["active_total"] > most * views * 5 // 4 + 4096  # beyond the guess at the records
        most = max(most, max(sg["active_per_view"]))
        assert np.array_equal(r.debug("tile_vals"), f.debug("tile_vals"))
        _close_grads(r.backward(dl), f.backward(dl))


def test_a_refused_render_writes_no_output():
    """A view over the instance cap is a capacity error that leaves its outputs as
    they were, also when earlier renders let the stages be enqueued before the
    counts are known: with and without the tile queue, for images, flow and the
    no-allocation render."""
    from paper_2310_10642_amd import g4d
    sc = _big_splat_scene(93, 3000, grow=0.5, sh=1, to=1, mu_log_t=1.0)
    r, _ = PT.gpu_setup(sc)
    cam = scenegen.look_at_camera((0.3, 0.1, 3.5), 150, 110)
    calls = (lambda out: r.render([cam], [0.5], out=out),
             lambda out: r.render_flow([cam], [0.5], 0.1, out=out[0][:2 * 150 * 110]),
             lambda out: r.render_noalloc([cam], [0.5], out))
    ref = [x.clone() for x in r.render([cam], [0.5])]
    need = r.stats()["instances"]
    for queue in (0, -1):
        r.set_tuning(g4d.G4D_TUNE_PERSISTENT_BLOCKS, queue)
        for call in calls:
            for cap in (1, need // 2, need - 1):
                out = [torch.full_like(x, 7.0) for x in ref]
                r.set_tuning(g4d.G4D_TUNE_ROUND_INSTANCES, cap)
                with pytest.raises(g4d.G4DError) as ei:
                    call(out)
                torch.cuda.synchronize()
                assert ei.value.status == g4d.G4D_ECAPACITY
                assert all(bool((x == 7.0).all()) for x in out), (queue, cap)
        r.set_tuning(g4d.G4D_TUNE_ROUND_INSTANCES, need)
        for a, b in zip(r.render([cam], [0.5]), ref):
            assert torch.equal(a, b)


def test_backward_clamps_the_alpha_of_very_long_needles():
    """Footprints thousands of pixels long and under one wide: in FP32 the quadratic
    form of such a record comes out positive for some pixels, so that an opacity
    of 0.985 gives alphas above the clamp at 0.99, and above 1. Three
    1920x1080 views in one launch (24480 tiles: one wave per tile) give the
    gradient lines of three launches of one view (8160 tiles: four waves per tile),
    whose products are the same value for value. The lines' position sums are
    then formed in FP64, and the colour sums are float32 sums of 256 terms a tile,
    as in test_backward_one_wave_per_tile. (The lines, not the primitives'
    gradients: those multiply the float32 rounding of a pair's dL/dSigma by the
    square of the long axis.)"""
    n = 200
    sc = scenegen.random_scene(95, n, sh_degree=1, t_order=1)
    sc.log_scales4[:] = np.float32([2.5, -8.0, -8.0, 3.0])
    th = 0.5 * np.random.default_rng(95).uniform(0, np.pi, n)
    q = np.stack([np.cos(th), np.sin(th), 0 * th, 0 * th], 1).astype(np.float32)
    sc.q_left[:], sc.q_right[:] = q, q          # a turn by 2 th in the image plane
    sc.means4[:, :3] *= np.float32(0.5)
    sc.opacity_logit[:] = np.float32(math.log(0.985 / 0.015))
    r, _ = PT.gpu_setup(sc)
    cams = [scenegen.look_at_camera((0.01 * v, 0.0, 4.0), 1920, 1080) for v in range(3)]
    times, k = [0.4, 0.5, 0.6], 3 * 1920 * 1080
    dl = torch.from_numpy(np.random.default_rng(96).uniform(-1, 1, 3 * k).astype(np.float32)).cuda()

    def lines(v0, v1):
        r.render(cams[v0:v1], times[v0:v1])
        r.backward(dl[k * v0:k * v1])
        out = np.zeros(((v1 - v0) * n, 16))
        out[r.debug("ids")] = r.debug("grad2d")
        return out

    got, want = lines(0, 3), np.concatenate([lines(v, v + 1) for v in range(3)])
    assert np.isfinite(got).all()
    for col in range(9):
        assert np.linalg.norm(got[:, col] - want[:, col]) <= 3e-5 * np.linalg.norm(want[:, col]), col


@pytest.mark.parametrize("front", [1, 2, 3, 4])
def test_emission_of_records_without_a_tile(front):
    """Active records whose alpha-floor ellipse lies between the pixel centres of
    two tiles have no instance: blocks of 64 such records behind `front` instances, so that
    their place in the output is and is not a multiple of four. Image and lists
    are those of the scene without them."""
    cam = scenegen.look_at_camera((0.0, 0.0, 4.0), 64, 48)
    rng = np.random.default_rng(97)
    n, m = 200, front + 5
    z = np.concatenate([np.linspace(1.0, 1.2, front), np.linspace(2.0, 3.0, n), np.linspace(4.0, 4.5, 5)])
    u = np.concatenate([rng.uniform(4, 12, front), 16.0 + rng.uniform(-0.3, 0.3, n), rng.uniform(20, 28, 5)])
    v = np.concatenate([rng.uniform(4, 12, front), rng.uniform(2, 46, n), rng.uniform(20, 28, 5)])
    sc = scenegen.random_scene(98, n + m, sh_degree=1, t_order=1)
    sc.q_left[:], sc.q_right[:] = np.float32([1, 0, 0, 0]), np.float32([1, 0, 0, 0])
    sc.log_scales4[:] = np.float32([-9.0, -9.0, -9.0, 3.0])
    sc.means4[:] = np.stack([(u - 32) * z / cam.fx, (24 - v) * z / cam.fy, 4 - z, 0 * z + 0.5], 1)
    o = 1.0001 / 255
    sc.opacity_logit[:] = np.float32(2.0)
    sc.opacity_logit[front:front + n] = np.float32(math.log(o / (1 - o)))
    r, _ = PT.gpu_setup(sc)
    got = r.render([cam], [0.5])
    st = r.stats()
    assert st["active_total"] == n + m and st["instances"] == m
    keep = np.r_[:front, front + n:front + n + 5]
    for a in ("means4", "log_scales4", "q_left", "q_right", "opacity_logit", "coeffs"):
        setattr(sc, a, getattr(sc, a)[keep])
    f, _ = PT.gpu_setup(sc)
    for a, b in zip(got, f.render([cam], [0.5])):
        assert torch.equal(a, b)
    assert f.stats()["instances"] == m and np.array_equal(r.debug("ranges"), f.debug("ranges"))


def test_capture_after_a_synchronous_render():
    """The scratch of a call depends on its shape, not on the counts that earlier
    calls saw: a sync-free render is captured right after a synchronous one of the
    same shape, whose counts let the depth sort take the chained passes for the
    first time (2.1M pairs, few of them active), and its replays give its image."""
    from paper_2310_10642_amd import g4d
    sc = scenegen.random_scene(101, 262145, sh_degree=0, t_order=0, mu_log_t=-4.0)
    r, _ = PT.gpu_setup(sc)
    cams = [scenegen.ring_camera(0.5 * v, 96, 64) for v in range(8)]
    times = [0.1 * v for v in range(8)]
    ref = r.render(cams, times)
    assert 0 < r.stats()["active_total"] * 5 // 4 + 4096 < 3 << 18
    out = [torch.empty_like(x) for x in ref]
    r.set_tuning(g4d.G4D_TUNE_SYNC_FREE, 1)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        r.render(cams, times, out=out)
    for _ in range(3):
        for t in out:
            t.fill_(float("nan"))
        x = torch.randn(512, 512, device="cuda")
        _ = float((x @ x).sum())               # eager work and a synchronisation
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(out, ref):
            assert torch.equal(a, b)
    del graph


def test_resident_workgroups_of_each_kernel():
    """G4D_TUNE_PERSISTENT_BLOCKS = -1 sizes each rasteriser's grid by that
    kernel's own residency, whatever was launched before: after one view (5440
    tiles: workgroups of 256 threads, 5 to a CU in the backward) eight views (one wave per
    tile, 16 to a CU) hold the whole device. Results are the same; the eight views'
    backward takes 1.3 times the time of one workgroup per tile (2.4 on the
    first kernel's grid)."""
    from paper_2310_10642_amd import g4d
    wl = scenegen.bench_workload(8)
    r, _ = PT.gpu_setup(wl.scene)
    times = [float(x) for x in wl.times]
    dl = torch.from_numpy(np.random.default_rng(58).uniform(-1, 1, 8 * 3 * 1352 * 1014).astype(np.float32)).cuda()
    ms, out = {}, {}
    for queue in (0, -1):
        r.set_tuning(g4d.G4D_TUNE_PERSISTENT_BLOCKS, queue)
        for views in (1, 8):
            best = float("inf")
            for _ in range(6):
                img = r.render(wl.cameras[:views], times[:views])
                r.stage_timing(True)
                grads = r.backward(dl[:img[0].numel()])
                best = min(best, r.stage_times()["raster_bwd"][0])
                r.stage_timing(False)
            out[queue, views], ms[queue, views] = (img, grads), best
    for views in (1, 8):
        for a, b in zip(out[0, views][0], out[-1, views][0]):
            assert torch.equal(a, b)
        _close_grads(out[-1, views][1], out[0, views][1])
    _say(f"  {ms}")
    assert ms[-1, 8] <= 1.8 * ms[0, 8]


@pytest.mark.parametrize("blocks", [1, 4, 512, 2048])
def test_large_tile_sort_on_any_grid(blocks):
    """G4D_TUNE_SORT_BLOCKS sizes the wide workgroups' grid of the tile sort from
    2^24 instances on too (1, 4, 512 and 818 workgroups here); the image and the
    tile lists are those of the default."""
    from paper_2310_10642_amd import g4d
    r, _ = PT.gpu_setup(_big_splat_scene(71, 3300, grow=3.0, sh=1, to=1, mu_log_t=1.0))
    cams = [scenegen.ring_camera(0.3 * v, 512, 512) for v in range(6)]
    times = [0.1 * v for v in range(6)]
    one = r.render(cams, times)
    vals = r.debug("tile_vals")
    assert r.stats()["rounds"] == 1 and len(vals) >= 1 << 24
    r.set_tuning(g4d.G4D_TUNE_SORT_BLOCKS, blocks)
    for a, b in zip(one, r.render(cams, times)):
        assert torch.equal(a, b)
    assert np.array_equal(vals, r.debug("tile_vals"))


def test_counts_that_come_back():
    """The guess at the counts forgets a crowded render: after 40 sparse ones the
    next crowded one is beyond it again, and the images, statistics and lists are
    those of a new context."""
    sc = _near_and_far_scene(103, 300, 20000)
    r, _ = PT.gpu_setup(sc)
    cams = [scenegen.look_at_camera((0.2, 0.1, 4.0), 160, 120)]
    for t in [0.9] + [0.1] * 40 + [0.9, 0.1, 0.9]:
        got = r.render(cams, [t])
        f, _ = PT.gpu_setup(sc)
        for a, b in zip(got, f.render(cams, [t])):
            assert torch.equal(a, b), t
        assert r.stats() == f.stats() and np.array_equal(r.debug("tile_vals"), f.debug("tile_vals"))


@pytest.mark.parametrize("t_cull", [0.0, 1e-30, 0.05, 0.999, 1.0])
@pytest.mark.parametrize("t", [0.0, 1000.5, -3e7])
def test_temporal_filter_against_the_oracle(t, t_cull, monkeypatch):
    """The pairs that pass p(t) >= t_cull are the FP64 definition's: primitives from
    1e-4 of the boundary to ten times it away, temporal scales from e^-80 to e^40
    (squares that underflow and overflow single precision), at times near and far
    from zero, half of them with quaternions of any orientation and of norms from 2^-60
    to 2^60. Left out: pairs within 1e-6 of the boundary, or whose rectangle
    FP64 rounding decides."""
    from paper_2310_10642_amd import g4d
    n, rng = 6000, np.random.default_rng(107)
    sc = scenegen.random_scene(107, n, sh_degree=0, t_order=0)
    half = n // 2
    sc.q_left[:half], sc.q_right[:half] = np.float32([1, 0, 0, 0]), np.float32([1, 0, 0, 0])
    sc.log_scales4[:half, 3] = rng.uniform(-80, 40, half).astype(np.float32)
    sc.log_scales4[half:, 3] = rng.uniform(-6, 2, n - half).astype(np.float32)
    sc.q_left[half:] *= (2.0 ** rng.integers(-60, 61, (n - half, 1))).astype(np.float32)
    sc.q_right[half:] *= (2.0 ** rng.integers(-60, 61, (n - half, 1))).astype(np.float32)
    sc.means4[:, :3] *= np.float32(0.3)
    p = O.params_from_scene(sc)
    s44 = O.covariance_4d(p["log_scales4"], p["q_left"], p["q_right"])[:, 3, 3].numpy()
    edge = np.sqrt(-2.0 * np.log(min(max(t_cull, 1e-300), 0.999)) * s44)
    off = rng.choice([0.0, 0.9, 0.999, 0.9999, 1.0001, 1.001, 1.1, 10.0], n) * rng.choice([-1.0, 1.0], n)
    with np.errstate(over="ignore"):
        sc.means4[:, 3] = np.clip(t + off * edge, -3e38, 3e38).astype(np.float32)
    monkeypatch.setitem(O.CONVENTIONS, "t_cull", PT.f32(t_cull))
    cam = scenegen.look_at_camera((0.3, 0.2, 3.5), 96, 80)
    pre = O.preprocess(O.params_from_scene(sc), O.to_ocamera(cam), PT.f32(t), 0, 0)
    pt, rects = pre["pt"].numpy(), (pre["rect_sure"].numpy(), pre["rect_maybe"].numpy(), pre["rect"].numpy())
    full = [(r[:, 2] > r[:, 0]) & (r[:, 3] > r[:, 1]) for r in rects]
    kept = pt >= PT.f32(t_cull)
    sure = (np.abs(pt - PT.f32(t_cull)) > 1e-6 * PT.f32(t_cull)) | (sc.means4[:, 3] == np.float32(t)) | (t_cull == 0)
    sure &= np.isfinite(pt) & (~kept | (full[0] == full[1]) | (t_cull in (0.0, 1.0)))  # (there the oracle is never sure)
    want = kept & full[2] & (pre["z"].numpy() > O.CONVENTIONS["near"])
    r = g4d.Renderer(0, 0, t_cull=t_cull)
    params = [torch.from_numpy(np.ascontiguousarray(a)).cuda()
              for a in (sc.means4, sc.log_scales4, sc.q_left, sc.q_right, sc.opacity_logit, sc.coeffs)]
    r.set_primitives(*params)
    r.set_tuning(g4d.G4D_TUNE_ELLIPSE_CULL, 0)
    r.render([cam], [t])
    got = np.zeros(n, bool)
    got[r.debug("ids")] = True
    _say(f"  t {t} t_cull {t_cull}: {int(got.sum())} active, {int((want & sure).sum())} surely, "
         f"{int((~sure).sum())} left out")
    assert sure.sum() > 0.7 * n and (want & sure).sum() > 100
    assert np.array_equal(got[sure], want[sure]), np.flatnonzero(sure & (got != want))[:10]


@pytest.mark.parametrize("views", [1, 300, 1710])
def test_gradients_of_records_without_opacity(views):
    """With the ellipse cull off and t_cull = 0, records whose opacity times p(t)
    underflows to zero are binned. They blend nowhere: their gradients are 0, not
    0 / 0, whatever shares their batch, and the others' those of the cull, in each of
    the three backward kernels (12, 3600 and 20520 tiles)."""
    from paper_2310_10642_amd import g4d
    sc = _big_splat_scene(109, 301, grow=0.4, sh=1, to=1, mu_log_t=-5.0)
    sc.means4[::3, 3] = np.float32(0.5)
    r = g4d.Renderer(1, 1, t_cull=0.0)
    params = [torch.from_numpy(np.ascontiguousarray(a)).cuda()
              for a in (sc.means4, sc.log_scales4, sc.q_left, sc.q_right, sc.opacity_logit, sc.coeffs)]
    r.set_primitives(*params)
    cams = [scenegen.ring_camera(0.01 * v, 61, 45) for v in range(views)]
    dl = torch.from_numpy(np.random.default_rng(110).uniform(-1, 1, views * 3 * 61 * 45).astype(np.float32)).cuda()
    want = [x.clone() for x in (r.render(cams, [0.5] * views)[0], *r.backward(dl))]
    few = r.stats()["active_total"]
    r.set_tuning(g4d.G4D_TUNE_ELLIPSE_CULL, 0)
    rgb = r.render(cams, [0.5] * views)[0]
    assert torch.equal(rgb, want[0]) and r.stats()["active_total"] > few
    assert (r.debug("records")[:, 3] == 0).any()
    _close_grads(r.backward(dl), want[1:])
