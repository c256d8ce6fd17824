"""GPU parity of the HIP path against the FP64 oracle (through the C ABI).

Bar: bit-exact projection decisions, pair lists, tile ranges, index map and
M_unstable; <= 1e-4 normwise relative error on colour, depth, transmission
and every gradient tensor."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from rtg_synth import make_config, random_upstream
from tests.gpu_helpers import (T_EPS, assert_parity, compare_forward, dev_mask, dev_params, dev_poses, fmt_stats,
                               gpu_forward, grad_stats, need_gpu, oracle_forward, oracle_grads, rel_err, ws_view)
from tests.scenes_small import (edge_on_surfels, footprint_condition, identity_pose, random_pose, random_scene,
                                small_cam, scene_from)

pytestmark = pytest.mark.gpu

TOL = 1e-4


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()
    from paper_2404_19706_amd import lib
    lib()
    yield


def _rast(cam, n, frames=1, **kw):
    from paper_2404_19706_amd import Rasterizer
    return Rasterizer(cam, n, frames, **kw)


def _two_pose_scene(seed, n=1500, cam=None):
    rng = np.random.default_rng(seed)
    pose_a, Rg, tg = random_pose(rng)
    target = tg + 2.0 * Rg[:, 2]
    from rtg_synth import look_at
    pose_b = look_at(tg + 0.15 * Rg[:, 0], target, up=-Rg[:, 1])
    sc = random_scene(rng, n, centre=target, spread=0.6, unstable_frac=0.6)
    return sc, np.stack([pose_a, pose_b])


def _check_pairs(rast, ws, P, recs, mask, F, N, g):
    """Per-tile pair counts, starts and sorted Gaussian lists equal the
    oracle's binning."""
    b = orc.bin_pairs(P, recs, mask)
    nt = b["tile_active"].shape[1]
    tend = ws_view(rast, ws, "tile_end", torch.int32, F * nt).cpu().numpy()
    start = ws_view(rast, ws, "tile_start", torch.int32, F * nt).cpu().numpy()
    npairs = tend - start
    K = int(npairs.sum())
    assert K == b["K"] == g["status"]["pairs"]
    pairs = ws_view(rast, ws, "pairs", torch.int32, K).cpu().numpy().astype(np.int64)
    cnt = np.bincount(b["frame"] * nt + b["tile"], minlength=F * nt)
    assert np.array_equal(cnt, npairs)
    nz = cnt > 0
    assert np.array_equal(start[nz], np.concatenate([[0], np.cumsum(cnt)[:-1]])[nz])
    got_gid = pairs - (np.repeat(np.arange(F * nt), cnt) // nt) * N
    assert np.array_equal(got_gid, b["gid"])


# ------------------------------------------------------------ decisions

@pytest.mark.parametrize("tile,size,flat", [((16, 16), (100, 75), 0.0), ((8, 8), (100, 75), 0.0),
                                            ((32, 8), (100, 75), 0.0), ((8, 8), (1030, 1030), 0.0),
                                            ((8, 8), (100, 75), 1e-6), ((32, 8), (400, 300), 1e-9)])
def test_projection_and_binning_bit_exact(tile, size, flat):
    """Ragged tiles on both axes; the 1030x1030 case has 129 x 129 tiles of
    8x8, more than one binning block's LDS chunk of tiles.  The flat cases
    make every Gaussian a surfel of that thickness, so surfels seen near
    edge-on give needle footprints for the pair thinning (condition numbers
    above 1e5; at 1e-9 one binary32 conic is not positive definite)."""
    W, H = size
    cam = small_cam(W, H, 90.0 * W / 100.0)
    sc, poses = _two_pose_scene(1, n=1200)
    if flat:
        sc["scale"][:, 2] = flat
    F, N = poses.shape[0], len(sc["pos"])
    rng = np.random.default_rng(2)
    mask = (rng.random((F, H, W)) < 0.3).astype(np.uint8)
    mask[1, H // 4:H // 2, W // 3:4 * W // 5] = 1
    rast = _rast(cam, N, F, tile_w=tile[0], tile_h=tile[1])
    g = gpu_forward(rast, sc, poses, mask)
    P = orc.make_params(cam, tile=tile)
    recs = orc.project(P, sc, poses)
    ws = g["ws"]
    vis = ws_view(rast, ws, "vis", torch.int32, N).cpu().numpy().view(np.uint32)
    hot = ws_view(rast, ws, "hot", torch.float32, 16 * F * N).cpu().numpy().reshape(F, N, 16)
    zk = ws_view(rast, ws, "zkey", torch.float32, F * N).cpu().numpy().reshape(F, N)
    rect = ws_view(rast, ws, "rect", torch.int16, 4 * F * N).cpu().numpy().reshape(F, N, 4)
    for f in range(F):
        ov = recs["visible"][f] != 0
        gv = ((vis >> f) & 1) != 0
        assert np.array_equal(ov, gv), f
        r = recs[f][ov]
        h = hot[f][ov]
        assert np.array_equal(h[:, 0].view(np.uint32), r["mu32"][:, 0].view(np.uint32))
        assert np.array_equal(h[:, 1].view(np.uint32), r["mu32"][:, 1].view(np.uint32))
        assert np.array_equal(h[:, 2].view(np.uint32), r["conic32"][:, 0].view(np.uint32))
        assert np.array_equal(h[:, 3], 2.0 * r["conic32"][:, 1])
        assert np.array_equal(h[:, 4].view(np.uint32), r["conic32"][:, 2].view(np.uint32))
        assert np.array_equal(h[:, 6].view(np.uint32), r["tau32"].view(np.uint32))
        assert np.array_equal(zk[f][ov].view(np.uint32), r["z32"].view(np.uint32))
        assert np.array_equal(rect[f][ov].astype(np.int32), r["rect"])
    _check_pairs(rast, ws, P, recs, mask, F, N, g)


@pytest.mark.parametrize("tile", [(8, 8), (16, 16)])
def test_edge_on_surfels_bit_exact_decisions(tile):
    """Surfels seen edge-on (needle footprints, condition numbers up to
    1e10): rectangles, visibility, pair lists and the index map bit-exact,
    including the pixels that binary32 rounding of the decision form admits
    beyond the ellipse."""
    cam = small_cam()
    sc = edge_on_surfels(np.random.default_rng(5), 400)
    poses = identity_pose()
    N = len(sc["pos"])
    mask = np.ones((1, cam["height"], cam["width"]), np.uint8)
    rast = _rast(cam, N, 1, tile_w=tile[0], tile_h=tile[1])
    g = gpu_forward(rast, sc, poses, mask)
    P, recs, pix, out = oracle_forward(cam, sc, poses, mask, tile=tile)
    ws = g["ws"]
    vis = ws_view(rast, ws, "vis", torch.int32, N).cpu().numpy().view(np.uint32)
    rect = ws_view(rast, ws, "rect", torch.int16, 4 * N).cpu().numpy().reshape(N, 4)
    ov = recs["visible"][0] != 0
    assert np.array_equal(ov, (vis & 1) != 0)
    assert np.array_equal(rect[ov].astype(np.int32), recs[0]["rect"][ov])
    _check_pairs(rast, ws, P, recs, mask, 1, N, g)
    e = compare_forward(g, pix, out, recs)
    print("edge-on surfels", tile, fmt_stats(e))
    assert e["index_mismatch"] == 0


@pytest.mark.parametrize("band", [2, 3, 4, 6, 8])
def test_needle_footprint_values(band):
    """Value parity on needle footprints: surfels seen exactly edge-on with
    thickness chosen so that the footprint condition number kappa lies in
    about [10^band, 10^(band+1)].  Colour, depth, transmission and the
    gradients of a random upstream against the oracle at every pixel."""
    cam = small_cam()
    lo, hi = -1.0 - (band + 1) / 2.0, -1.0 - band / 2.0
    sc = edge_on_surfels(np.random.default_rng(40 + band), 300, thick_exp=(lo, hi), tilt_exp=None)
    poses = identity_pose()
    N = len(sc["pos"])
    mask = np.ones((1, cam["height"], cam["width"]), np.uint8)
    rast = _rast(cam, N, 1)
    g = gpu_forward(rast, sc, poses, mask)
    P, recs, pix, out = oracle_forward(cam, sc, poses, mask)
    kap = footprint_condition(recs)[0]
    kap = kap[np.isfinite(kap)]
    e = compare_forward(g, pix, out, recs)
    gC, gD = random_upstream(mask, seed=41)
    grads = rast.alloc_grads()
    C, D, T, I = g["tensors"]
    rast.backward_into(g["ws"], g["params"], dev_poses(poses), D, T, I,
                       torch.as_tensor(gC).cuda(), torch.as_tensor(gD).cuda(), grads)
    torch.cuda.synchronize()
    f, x, y = pix[:, 0], pix[:, 1], pix[:, 2]
    ref, gbnd = oracle_grads(P, recs, sc, poses, pix, gC[f, y, x], gD[f, y, x])
    e.update(grad_stats(grads, ref, sc["unstable"], gbnd))
    print("needle band 1e%d: kappa %.1e..%.1e (median %.1e), %d pixels with a list" %
          (band, kap.min(), kap.max(), np.median(kap), int((out["nlist"] > 0).sum())), fmt_stats(e), flush=True)
    assert e["index_mismatch"] == 0
    assert_parity(e)


# ------------------------------------------------------------ forward values

def test_forward_parity_c1():
    cfg = make_config("c1")
    cam, sc, poses = cfg["cam"], cfg["scene"], cfg["poses"]
    mask = np.ones((1, cam["height"], cam["width"]), np.uint8)
    rast = _rast(cam, len(sc["pos"]), 1)
    g = gpu_forward(rast, sc, poses, mask)
    _, recs, pix, out = oracle_forward(cam, sc, poses, mask)
    e = compare_forward(g, pix, out, recs)
    print("c1 forward errors", fmt_stats(e))
    assert e["index_mismatch"] == 0
    assert_parity(e)


def test_forward_masked_ragged_two_frames():
    cam = small_cam(100, 75, 90.0)
    sc, poses = _two_pose_scene(3, n=2000)
    rng = np.random.default_rng(4)
    mask = (rng.random((2, 75, 100)) < 0.15).astype(np.uint8)
    rast = _rast(cam, len(sc["pos"]), 2)
    g = gpu_forward(rast, sc, poses, mask)
    _, recs, pix, out = oracle_forward(cam, sc, poses, mask)
    e = compare_forward(g, pix, out, recs)
    print("ragged masked errors", fmt_stats(e))
    assert e["index_mismatch"] == 0
    assert_parity(e)
    # unmasked pixels keep the caller's prefill
    off = mask == 0
    assert (g["color"][off] == 0).all() and (g["trans"][off] == 1).all()
    assert (g["depth"][off] == -1).all() and (g["index"][off] == -1).all()


def test_forward_bit_identical_across_tiles_and_queue_granularity():
    cfg = make_config("c1")
    cam, sc, poses = cfg["cam"], cfg["scene"], cfg["poses"]
    rng = np.random.default_rng(5)
    mask = (rng.random((1, cam["height"], cam["width"])) < 0.5).astype(np.uint8)
    ref = None
    for tile in [(16, 16), (8, 8), (32, 8)]:
        # (items_per_pop, static_share, forward's own items_per_pop and share)
        for sched in ((0, 0, -1, -1), (1, 0, -1, -1), (3, 0, -1, -1), (2, 50, 4, 50), (0, 0, 2, 30)):
            rast = _rast(cam, len(sc["pos"]), 1, tile_w=tile[0], tile_h=tile[1], items_per_pop=sched[0],
                         static_share=sched[1], fwd_items_per_pop=sched[2], fwd_static_share=sched[3])
            g = gpu_forward(rast, sc, poses, mask)
            cur = [g[k] for k in ("color", "depth", "trans", "index")]
            if ref is None:
                ref = cur
            else:
                for a, b in zip(cur, ref):
                    assert np.array_equal(a.view(np.uint32) if a.dtype != np.int32 else a,
                                          b.view(np.uint32) if b.dtype != np.int32 else b)


@pytest.mark.parametrize("lanes,tile", [(4, (16, 16)), (32, (16, 16)), (32, (8, 8)), (8, (32, 8))])
def test_straggler_path_is_bit_identical(lanes, tile):
    """The forward compositing kernel switches a pack's last few live
    pixels to the straggler path (each walks the rest of its list alone,
    one entry per lane); with the switch forced early (any remaining entry)
    the render equals that of the pack path bit for bit, the gradients
    (whose backward reads the render's per-pixel list ends) equal its
    gradients up to the order of the float atomic sums, and both match the
    oracle."""
    cam = small_cam(100, 75, 90.0)
    sc, poses = _two_pose_scene(41, n=4000)
    rng = np.random.default_rng(42)
    mask = (rng.random((2, 75, 100)) < 0.5).astype(np.uint8)
    N = len(sc["pos"])
    kw = dict(tile_w=tile[0], tile_h=tile[1])
    runs = []
    for sl in (0, lanes):
        rast = _rast(cam, N, 2, straggler_lanes=sl, straggler_rest=1, **kw)
        g = gpu_forward(rast, sc, poses, mask)
        gC, gD = random_upstream(mask, seed=43)
        grads = rast.alloc_grads()
        C, D, T, I = g["tensors"]
        rast.backward_into(g["ws"], g["params"], dev_poses(poses), D, T, I, torch.as_tensor(gC).cuda(),
                           torch.as_tensor(gD).cuda(), grads)
        torch.cuda.synchronize()
        runs.append((g, [grads[k].cpu().numpy() for k in sorted(grads)]))
    (g0, gr0), (g1, gr1) = runs
    for k in ("color", "depth", "trans", "index"):
        a, b = g0[k], g1[k]
        assert np.array_equal(a.view(np.uint32) if a.dtype != np.int32 else a,
                              b.view(np.uint32) if b.dtype != np.int32 else b), k
    for a, b in zip(gr0, gr1):
        np.testing.assert_allclose(a, b, rtol=1e-5, atol=1e-6 * (np.abs(a).max() + 1e-30))
    _, recs, pix, out = oracle_forward(cam, sc, poses, mask, tile=tile)
    e = compare_forward(g1, pix, out, recs)
    assert e["index_mismatch"] == 0
    assert_parity(e)
    errs = _grad_parity(cam, sc, poses, mask, seed=43, straggler_lanes=lanes, straggler_rest=1, **kw)
    print("straggler path gradient errors", lanes, tile, fmt_stats(errs))
    assert_parity(errs)


@pytest.mark.parametrize("cap", [64, 1, 200])
def test_long_list_sort_path_matches_lds_path(cap):
    """Lists above sort_cap are sorted in LDS runs of a power of two >= 2 cap
    (>= 64) and merged; the pair lists must equal the one-pass LDS sort's."""
    cfg = make_config("c1")
    cam, sc, poses = cfg["cam"], cfg["scene"], cfg["poses"]
    mask = np.ones((1, cam["height"], cam["width"]), np.uint8)
    r1, r2 = _rast(cam, len(sc["pos"]), 1), _rast(cam, len(sc["pos"]), 1, sort_cap=cap)
    g1 = gpu_forward(r1, sc, poses, mask)
    g2 = gpu_forward(r2, sc, poses, mask)
    assert g2["status"]["big_tiles"] > 0 and g1["status"]["big_tiles"] == 0
    K = g1["status"]["pairs"]
    assert g2["status"]["pairs"] == K
    p1 = ws_view(r1, g1["ws"], "pairs", torch.int32, K).cpu().numpy()
    p2 = ws_view(r2, g2["ws"], "pairs", torch.int32, K).cpu().numpy()
    assert np.array_equal(p1, p2)
    for k in ("color", "depth", "trans", "index"):
        assert np.array_equal(g1[k], g2[k])


def test_long_list_sort_with_tight_capacity():
    """With the pair capacity equal to the pair count the long-list sort runs
    on its smallest grid (capacity / (sort_cap + 1) + 1 workgroups); every
    listed tile is still sorted."""
    cfg = make_config("c1")
    cam, sc, poses = cfg["cam"], cfg["scene"], cfg["poses"]
    mask = np.ones((1, cam["height"], cam["width"]), np.uint8)
    r1 = _rast(cam, len(sc["pos"]), 1)
    g1 = gpu_forward(r1, sc, poses, mask)
    K = g1["status"]["pairs"]
    r2 = _rast(cam, len(sc["pos"]), 1, max_pairs=K, sort_cap=64)
    g2 = gpu_forward(r2, sc, poses, mask)
    assert g2["status"]["big_tiles"] > 0 and not g2["status"]["overflow"] and g2["status"]["pairs"] == K
    p1 = ws_view(r1, g1["ws"], "pairs", torch.int32, K).cpu().numpy()
    p2 = ws_view(r2, g2["ws"], "pairs", torch.int32, K).cpu().numpy()
    assert np.array_equal(p1, p2)
    for k in ("color", "depth", "trans", "index"):
        assert np.array_equal(g1[k], g2[k])


@pytest.mark.parametrize("cap", [0, 100])
def test_sort_paths_bit_exact(cap):
    """Per-tile lists from 1 to ~730 pairs: with the default cap the one-wave
    rank sort (<= 64 and <= 256 keys) and the workgroup LDS bitonic sort
    both run; with cap 100 every list above it takes the run sort (bitonic over 1024
    threads) plus merge rounds.  The lists must equal the oracle's."""
    cam = small_cam(96, 72, 80.0)
    sc, poses = _two_pose_scene(3, n=3000)
    F, N = poses.shape[0], len(sc["pos"])
    mask = np.ones((F, 72, 96), np.uint8)
    rast = _rast(cam, N, F, tile_w=16, tile_h=16, **({"sort_cap": cap} if cap else {}))
    g = gpu_forward(rast, sc, poses, mask)
    P = orc.make_params(cam, tile=(16, 16))
    recs = orc.project(P, sc, poses)
    nt = 6 * 5   # 16x16 tiles over 96x72
    ws = g["ws"]
    tend = ws_view(rast, ws, "tile_end", torch.int32, F * nt).cpu().numpy()
    tstart = ws_view(rast, ws, "tile_start", torch.int32, F * nt).cpu().numpy()
    n = tend - tstart
    if cap:
        assert g["status"]["big_tiles"] > 0 and n.max() > 2 * 256
    else:
        assert g["status"]["big_tiles"] == 0
        assert ((n > 64) & (n <= 256)).any() and (n > 256).any() and ((n > 0) & (n <= 64)).any()
    _check_pairs(rast, ws, P, recs, mask, F, N, g)


@pytest.mark.parametrize("cap", [0, 400, 1000])
def test_register_sort_sizes_bit_exact(cap):
    """A dense two-frame scene, per-tile lists from a few to ~4800 pairs.
    Default cap: the one-wave rank sort, LDS steps at 512 keys, the
    register-resident bitonic sort at 1024, 2048 and 4096 keys, and lists
    above 4096 as 4096-key run sorts plus a merge.  Caps 400 and 1000: run
    sorts of 1024 and 2048 keys (the power of two >= 2 cap) plus merges.
    The lists must equal the oracle's."""
    cam = small_cam(96, 72, 80.0)
    sc, poses = _two_pose_scene(3, n=20000)
    F, N = poses.shape[0], len(sc["pos"])
    mask = np.ones((F, 72, 96), np.uint8)
    rast = _rast(cam, N, F, tile_w=16, tile_h=16, **({"sort_cap": cap} if cap else {}))
    g = gpu_forward(rast, sc, poses, mask)
    P = orc.make_params(cam, tile=(16, 16))
    recs = orc.project(P, sc, poses)
    nt = 6 * 5
    ws = g["ws"]
    tend = ws_view(rast, ws, "tile_end", torch.int32, F * nt).cpu().numpy()
    tstart = ws_view(rast, ws, "tile_start", torch.int32, F * nt).cpu().numpy()
    n = tend - tstart
    for lo, hi in ((0, 256), (256, 512), (512, 1024), (1024, 2048), (2048, 4096), (4096, 1 << 30)):
        assert ((n > lo) & (n <= hi)).any(), (lo, hi)
    assert g["status"]["big_tiles"] > 0
    _check_pairs(rast, ws, P, recs, mask, F, N, g)


@pytest.mark.parametrize("cap", [0, 100])
def test_tile_ranges_over_many_chunks(cap):
    """Eight frames of 40 x 30 tiles (9,600 (frame, tile)s, three chunks of
    4096, so the chunk-parallel range and item pass runs), with and without
    long lists: pair lists equal the oracle's, the item count is that of the
    packs, and the render is bit-identical to the frames rendered one plan
    each (one chunk)."""
    cam = small_cam(320, 240, 280.0)
    rng = np.random.default_rng(33)
    pose_a, Rg, tg = random_pose(rng)
    target = tg + 2.0 * Rg[:, 2]
    from rtg_synth import look_at
    F = 8
    poses = np.stack([look_at(tg + 0.05 * k * Rg[:, 0], target, up=-Rg[:, 1]) for k in range(F)])
    sc = random_scene(rng, 4000, centre=target, spread=0.6)
    N = len(sc["pos"])
    mask = (rng.random((F, 240, 320)) < rng.uniform(0.2, 0.9, (F, 1, 1))).astype(np.uint8)
    kw = dict(tile_w=8, tile_h=8, **({"sort_cap": cap} if cap else {}))
    rast = _rast(cam, N, F, **kw)
    g = gpu_forward(rast, sc, poses, mask)
    P = orc.make_params(cam, tile=(8, 8))
    recs = orc.project(P, sc, poses)
    _check_pairs(rast, g["ws"], P, recs, mask, F, N, g)
    npx = mask.reshape(F, 30, 8, 40, 8).sum((2, 4))
    assert g["status"]["items"] == int(((npx + 63) // 64).sum())
    assert g["status"]["pixels"] == int(mask.sum())
    if cap:
        assert g["status"]["big_tiles"] > 0
    for f in range(F):
        r1 = _rast(cam, N, 1, **kw)
        g1 = gpu_forward(r1, sc, poses[f:f + 1], mask[f:f + 1])
        for k in ("color", "depth", "trans", "index"):
            assert np.array_equal(g[k][f], g1[k][0]), (f, k)


def test_pair_staging_overflow_gives_the_same_lists():
    """The counting pass stages every pair it finds; a binning block whose
    staging region overflows enumerates its pairs a second time instead.
    With the default capacity nothing falls back; with regions of one entry
    every block with a pair does, and with regions of the median block's
    pair count only the blocks above it (both paths in one binning).  The
    pair lists equal the oracle's and the renders are bit-identical.  Here
    every binning block (256 Gaussians of one frame) has a region of its
    own."""
    W, H = 400, 300
    cam = small_cam(W, H, 90.0 * W / 100.0)
    sc, poses = _two_pose_scene(1, n=1200)
    F, N = poses.shape[0], len(sc["pos"])
    rng = np.random.default_rng(2)
    mask = (rng.random((F, H, W)) < 0.3).astype(np.uint8)
    P = orc.make_params(cam, tile=(8, 8))
    recs = orc.project(P, sc, poses)
    b = orc.bin_pairs(P, recs, mask)
    per_block = np.bincount(b["frame"] * 5 + b["gid"] // 256, minlength=F * 5)
    with_pairs = int((per_block > 0).sum())
    med = int(np.median(per_block))
    above = int((per_block > med).sum())
    assert 0 < above < with_pairs
    ref = None
    restaged = {}
    for cap in (0, 1, med):
        rast = _rast(cam, N, F, tile_w=8, tile_h=8, **({"stage_cap": cap} if cap else {}))
        g = gpu_forward(rast, sc, poses, mask)
        restaged[cap] = g["status"]["restaged_blocks"]
        _check_pairs(rast, g["ws"], P, recs, mask, F, N, g)
        if ref is None:
            ref = g
        else:
            for k in ("color", "depth", "trans", "index"):
                assert np.array_equal(ref[k], g[k]), (cap, k)
    assert restaged == {0: 0, 1: with_pairs, med: above}, restaged


# ------------------------------------------------------------ edge cases

def test_empty_mask_and_all_culled():
    cfg = make_config("c1")
    cam, sc, poses = cfg["cam"], cfg["scene"], cfg["poses"]
    rast = _rast(cam, len(sc["pos"]), 1)
    g = gpu_forward(rast, sc, poses, np.zeros((1, cam["height"], cam["width"]), np.uint8))
    assert g["status"]["pixels"] == 0 and g["status"]["pairs"] == 0 and g["status"]["items"] == 0
    assert (g["trans"] == 1).all() and (g["index"] == -1).all()
    behind = dict(sc)
    behind["pos"] = sc["pos"] * np.array([1, 1, -1], np.float32)
    g = gpu_forward(rast, behind, poses, np.ones((1, cam["height"], cam["width"]), np.uint8))
    assert g["status"]["pairs"] == 0 and g["status"]["pixels"] == cam["width"] * cam["height"]
    assert (g["trans"] == 1).all() and (g["depth"] == -1).all() and (g["color"] == 0).all()


def test_zero_gaussians():
    cam = small_cam(40, 30, 40.0)
    from tests.scenes_small import scene_from
    sc = scene_from(np.zeros((0, 3)), np.zeros((0, 3)), np.zeros((0, 4)), np.zeros(0), np.zeros((0, 3)))
    rast = _rast(cam, 0, 1)
    g = gpu_forward(rast, sc, identity_pose(), np.ones((1, 30, 40), np.uint8))
    assert g["status"]["pairs"] == 0 and (g["trans"] == 1).all()


def test_pair_capacity_overflow_reports_and_renders_nothing():
    cfg = make_config("c1")
    cam, sc, poses = cfg["cam"], cfg["scene"], cfg["poses"]
    rast = _rast(cam, len(sc["pos"]), 1, max_pairs=100)
    g = gpu_forward(rast, sc, poses, np.ones((1, cam["height"], cam["width"]), np.uint8))
    from paper_2404_19706_amd._lib import RTG_E_CAPACITY
    assert g["status"]["status"] == RTG_E_CAPACITY and g["status"]["overflow"] == 1
    assert g["status"]["items"] == 0
    # every tile's pair range is left empty, so the sorts have nothing to do
    tw, th = rast.cfg.tile_w, rast.cfg.tile_h
    nt = -(-cam["width"] // tw) * -(-cam["height"] // th)
    tend = ws_view(rast, g["ws"], "tile_end", torch.int32, nt).cpu().numpy()
    tstart = ws_view(rast, g["ws"], "tile_start", torch.int32, nt).cpu().numpy()
    assert (tend == tstart).all()
    assert (g["trans"] == 1).all() and (g["index"] == -1).all()


def test_invalid_arguments_are_rejected_on_the_host():
    from paper_2404_19706_amd import RtgError
    cam = small_cam(40, 30, 40.0)
    with pytest.raises(RtgError):
        _rast(cam, 10, 1, tile_w=12, tile_h=12)
    with pytest.raises(RtgError):
        _rast(cam, 10, 33)
    rast = _rast(cam, 10, 1)
    ws = rast.new_workspace()
    from paper_2404_19706_amd._lib import lib as L, RTG_E_INVALID
    import ctypes
    assert L().rtg_bin(rast._plan, ctypes.c_void_p(ws.data_ptr() + 1), ctypes.c_void_p(ws.data_ptr()),
                       None) == RTG_E_INVALID
    assert L().rtg_render(rast._plan, ctypes.c_void_p(ws.data_ptr()), None, None, None, None, None) == RTG_E_INVALID


# ------------------------------------------------------------ M_unstable

def test_unstable_mask_bit_exact():
    cam = small_cam(100, 75, 90.0)
    sc, poses = _two_pose_scene(6, n=1500)
    rast = _rast(cam, len(sc["pos"]), 2)
    m = rast.unstable_mask(dev_params(sc), dev_poses(poses)).cpu().numpy()
    P = orc.make_params(cam)
    recs = orc.project(P, sc, poses)
    ref = orc.unstable_mask_image(P, recs, sc["unstable"])
    assert 0.05 < ref.mean() < 0.95
    assert np.array_equal(m, ref)


def test_filter50_renders_the_filtered_pixel_set():
    cam = small_cam(100, 75, 90.0)
    sc, poses = _two_pose_scene(7, n=800)
    rng = np.random.default_rng(8)
    mask = (rng.random((2, 75, 100)) < rng.uniform(0.3, 0.7, (2, 1, 1))).astype(np.uint8)
    rast = _rast(cam, len(sc["pos"]), 2, tile_filter50=1)
    g = gpu_forward(rast, sc, poses, mask)
    eff = orc.filter50(orc.make_params(cam), mask)
    assert 0 < eff.sum() < mask.sum()
    assert g["status"]["pixels"] == int(eff.sum())
    assert np.array_equal(g["index"] != -1, (g["index"] != -1) & (eff != 0))
    assert (g["trans"][eff == 0] == 1).all()


# ------------------------------------------------------------ backward

def _grad_parity(cam, sc, poses, mask, seed, **kw):
    N, F = len(sc["pos"]), poses.shape[0]
    rast = _rast(cam, N, F, **kw)
    g = gpu_forward(rast, sc, poses, mask)
    gC, gD = random_upstream(mask, seed=seed)
    grads = rast.alloc_grads()
    C, D, T, I = g["tensors"]
    rast.backward_into(g["ws"], g["params"], dev_poses(poses), D, T, I,
                       torch.as_tensor(gC).cuda(), torch.as_tensor(gD).cuda(), grads)
    torch.cuda.synchronize()
    P, recs, pix, out = oracle_forward(cam, sc, poses, mask)
    f, x, y = pix[:, 0], pix[:, 1], pix[:, 2]
    ref, gbnd = oracle_grads(P, recs, sc, poses, pix, gC[f, y, x], gD[f, y, x])
    return grad_stats(grads, ref, sc["unstable"], gbnd)


def test_backward_parity_single_frame():
    cfg = make_config("c1")
    cam, sc, poses = cfg["cam"], dict(cfg["scene"]), cfg["poses"]
    sc["unstable"] = (np.random.default_rng(9).random(len(sc["pos"])) < 0.5).astype(np.uint8)
    mask = np.ones((1, cam["height"], cam["width"]), np.uint8)
    errs = _grad_parity(cam, sc, poses, mask, seed=10)
    print("c1 gradient errors", fmt_stats(errs))
    assert_parity(errs)


def test_backward_parity_masked_two_frames_ragged():
    cam = small_cam(100, 75, 90.0)
    sc, poses = _two_pose_scene(11, n=1500)
    rng = np.random.default_rng(12)
    mask = (rng.random((2, 75, 100)) < 0.4).astype(np.uint8)
    errs = _grad_parity(cam, sc, poses, mask, seed=13, tile_w=8, tile_h=8)
    print("ragged two-frame gradient errors", fmt_stats(errs))
    assert_parity(errs)


def test_autograd_function_matches_direct_calls():
    from paper_2404_19706_amd import rasterize_masked
    cfg = make_config("c1")
    cam, sc, poses = cfg["cam"], cfg["scene"], cfg["poses"]
    mask = np.ones((1, cam["height"], cam["width"]), np.uint8)
    rast = _rast(cam, len(sc["pos"]), 1)
    params = [p.clone().requires_grad_(True) if p.dtype == torch.float32 else p for p in dev_params(sc)]
    C, D, T, I = rasterize_masked(*params, dev_poses(poses), dev_mask(mask), rast)
    gC, gD = random_upstream(mask, seed=14)
    (C * torch.as_tensor(gC).cuda()).sum().add((D * torch.as_tensor(gD).cuda()).sum()).backward()
    g = gpu_forward(rast, sc, poses, mask)
    grads = rast.alloc_grads()
    rast.backward_into(g["ws"], g["params"], dev_poses(poses), *g["tensors"][1:],
                       torch.as_tensor(gC).cuda(), torch.as_tensor(gD).cuda(), grads)
    for p, k in zip(params[:5], ("pos", "scale", "rot", "opacity", "color")):
        assert rel_err(p.grad.cpu().numpy(), grads[k].cpu().numpy()) < 1e-6


# ------------------------------------------------------------ harness

def test_l1_loss_and_upstream_match_oracle():
    cfg = make_config("c1")
    cam, sc, poses = cfg["cam"], cfg["scene"], cfg["poses"]
    rng = np.random.default_rng(15)
    mask = (rng.random((1, cam["height"], cam["width"])) < 0.6).astype(np.uint8)
    rast = _rast(cam, len(sc["pos"]), 1)
    g = gpu_forward(rast, sc, poses, mask)
    C, D, T, I = g["tensors"]
    Cgt = torch.rand_like(C)
    Dgt = torch.where(torch.rand_like(D) < 0.1, torch.zeros_like(D), torch.rand_like(D) * 3)
    dC = torch.zeros_like(C)
    dD = torch.zeros_like(D)
    loss = torch.zeros(1, device="cuda")
    rast.loss_l1_into(g["ws"], C, D, Cgt, Dgt, dC, dD, loss)
    gc_ref, gd_ref, l_ref = orc.l1_upstream(C.cpu().numpy(), D.cpu().numpy(), Cgt.cpu().numpy(),
                                            Dgt.cpu().numpy(), mask)
    assert rel_err(dC.cpu().numpy(), gc_ref) < 1e-6
    assert rel_err(dD.cpu().numpy(), gd_ref) < 1e-6
    assert abs(float(loss) - l_ref) < 1e-5 * max(1.0, l_ref)


@pytest.mark.parametrize("tile,ipp", [((16, 16), 0), ((32, 8), 1)])
def test_fused_l1_backward_equals_separate_calls(tile, ipp):
    """rtg_backward_raster_l1 + rtg_backward_project_l1 give the loss value
    and parameter gradients of rtg_loss_l1 + rtg_backward_raster +
    rtg_backward_project up to float summation order; two frames, ragged
    masks, targets with invalid depths, weights other than one; twice in a
    row on the same projection (the per-wave sums are rewritten)."""
    cam = small_cam(100, 75, 90.0)
    sc, poses = _two_pose_scene(5, n=1500)
    rng = np.random.default_rng(16)
    mask = (rng.random((2, 75, 100)) < 0.5).astype(np.uint8)
    rast = _rast(cam, len(sc["pos"]), 2, tile_w=tile[0], tile_h=tile[1], items_per_pop=ipp)
    g = gpu_forward(rast, sc, poses, mask)
    C, D, T, I = g["tensors"]
    ws, params, dp = g["ws"], g["params"], dev_poses(poses)
    Cgt = torch.rand_like(C)
    Dgt = torch.where(torch.rand_like(D) < 0.1, torch.zeros_like(D), torch.rand_like(D) * 3)
    w_c, w_d = 0.7, 0.3
    dC, dD = torch.zeros_like(C), torch.zeros_like(D)
    loss_a = torch.zeros(1, device="cuda")
    rast.loss_l1_into(ws, C, D, Cgt, Dgt, dC, dD, loss_a, w_c=w_c, w_d=w_d)
    rast.backward_raster(ws, D, T, I, dC, dD)
    ga = rast.alloc_grads()
    rast.backward_project(ws, params, dp, ga)
    for _ in range(2):
        loss_b = torch.zeros(1, device="cuda")
        rast.backward_raster_l1(ws, C, D, T, I, Cgt, Dgt)
        gb = rast.alloc_grads()
        rast.backward_project_l1(ws, params, dp, gb, loss_b, w_c=w_c, w_d=w_d)
        torch.cuda.synchronize()
        assert abs(float(loss_b) - float(loss_a)) <= 1e-6 * abs(float(loss_a))
        # the scales enter after the float accumulation instead of before:
        # a few binary32 roundings per sum
        for k in ga:
            assert torch.count_nonzero(ga[k]) > 0, k
            assert rel_err(gb[k].cpu().numpy(), ga[k].cpu().numpy()) <= 1e-5, k


def test_adam_matches_oracle():
    from paper_2404_19706_amd import Rasterizer
    cam = small_cam(40, 30, 40.0)
    n = 300
    rng = np.random.default_rng(16)
    sc = random_scene(rng, n, unstable_frac=0.5)
    rast = Rasterizer(cam, n, 1)
    params = [p.clone() for p in dev_params(sc)]
    m = torch.zeros((n, 13), device="cuda")
    v = torch.zeros((n, 13), device="cuda")
    step = torch.zeros(1, dtype=torch.int32, device="cuda")
    lr = (1e-3, 2e-3, 1e-3, 1e-3)
    ref = {"pos": sc["pos"].astype(np.float64), "logs": np.log(sc["scale"].astype(np.float64)),
           "rot": sc["rot"].astype(np.float64), "color": sc["color"].astype(np.float64)}
    st = {k: (np.zeros_like(x), np.zeros_like(x)) for k, x in ref.items()}
    un = sc["unstable"]
    for it in range(1, 4):
        grads = {k: torch.as_tensor(rng.standard_normal(s).astype(np.float32)).cuda()
                 for k, s in (("pos", (n, 3)), ("scale", (n, 3)), ("rot", (n, 4)), ("color", (n, 3)))}
        s_now = params[1].cpu().numpy().astype(np.float64)
        rast.adam(params, grads, m, v, step, lr=lr, eps=1e-15)
        for k, lrk, gk in (("pos", lr[0], grads["pos"].cpu().numpy()),
                           ("logs", lr[1], s_now * grads["scale"].cpu().numpy()),
                           ("rot", lr[2], grads["rot"].cpu().numpy()),
                           ("color", lr[3], grads["color"].cpu().numpy())):
            ref[k], mm, vv = orc.adam_step(ref[k], gk, st[k][0], st[k][1], it, lrk, un, eps=1e-15)
            st[k] = (mm, vv)
    assert int(step.item()) == 3
    assert np.allclose(params[0].cpu().numpy(), ref["pos"], rtol=1e-5, atol=1e-6)
    assert np.allclose(params[1].cpu().numpy(), np.exp(ref["logs"]), rtol=1e-5, atol=1e-7)
    assert np.allclose(params[2].cpu().numpy(), ref["rot"], rtol=1e-5, atol=1e-6)
    assert np.allclose(params[4].cpu().numpy(), ref["color"], rtol=1e-5, atol=1e-6)
    assert np.array_equal(params[3].cpu().numpy(), sc["opacity"])


# ------------------------------------------------------------ binning bounds

def _gpu_pair_set(rast, ws, F, N, nt, K):
    tend = ws_view(rast, ws, "tile_end", torch.int32, F * nt).cpu().numpy().astype(np.int64)
    start = ws_view(rast, ws, "tile_start", torch.int32, F * nt).cpu().numpy().astype(np.int64)
    pairs = ws_view(rast, ws, "pairs", torch.int32, K).cpu().numpy().astype(np.int64)
    cnt = tend - start
    ft = np.repeat(np.arange(F * nt), cnt)
    pos = np.concatenate([np.arange(s, e) for s, e in zip(start, tend) if e > s]) if K else np.zeros(0, np.int64)
    gid = pairs[pos] - (ft // nt) * N
    return set((ft * N + gid).tolist())


@pytest.mark.parametrize("case,tile", [("c1", (16, 16)), ("ragged", (8, 8)), ("ragged", (32, 8)),
                                       ("edge_on", (16, 16))])
def test_pair_lists_lie_between_the_needed_and_the_plain_pairs(case, tile):
    """Independent of the pair-thinning rule both sides implement: every
    (frame, tile, Gaussian) pair the GPU bins is one the paper's plain rule
    would bin (the Gaussian's rectangle covers the tile, the tile has a
    masked pixel), and every pair a pixel needs (the Gaussian is in the list
    L(u) of a masked pixel u of that tile, from the oracle) is binned."""
    if case == "c1":
        cfg = make_config("c1")
        cam, sc, poses = cfg["cam"], cfg["scene"], cfg["poses"]
        mask = np.ones((1, cam["height"], cam["width"]), np.uint8)
    elif case == "ragged":
        cam = small_cam(100, 75, 90.0)
        sc, poses = _two_pose_scene(21, n=1500)
        mask = (np.random.default_rng(22).random((2, 75, 100)) < 0.3).astype(np.uint8)
    else:
        cam = small_cam()
        sc = edge_on_surfels(np.random.default_rng(23), 400)
        poses = identity_pose()
        mask = np.ones((1, cam["height"], cam["width"]), np.uint8)
    F, N = poses.shape[0], len(sc["pos"])
    rast = _rast(cam, N, F, tile_w=tile[0], tile_h=tile[1])
    g = gpu_forward(rast, sc, poses, mask)
    tw, th = tile
    tx, ty = -(-cam["width"] // tw), -(-cam["height"] // th)
    nt = tx * ty
    got = _gpu_pair_set(rast, g["ws"], F, N, nt, g["status"]["pairs"])
    P, recs, pix, _ = oracle_forward(cam, sc, poses, mask, tile=tile)
    # plain rule: rectangle tiles with a masked pixel
    act = np.zeros((F, ty, tx), bool)
    f_, x_, y_ = pix[:, 0], pix[:, 1], pix[:, 2]
    act[f_, y_ // th, x_ // tw] = True
    plain = set()
    for f in range(F):
        vis = np.nonzero(recs["visible"][f])[0]
        for i in vis:
            x0, x1, y0, y1 = recs["rect"][f, i]
            for b in range(y0 // th, y1 // th + 1):
                for a in range(x0 // tw, x1 // tw + 1):
                    if act[f, b, a]:
                        plain.add((f * nt + b * tx + a) * N + int(i))
    need = set()
    for (f, x, y), L in zip(pix, orc.pixel_lists(P, recs, pix)):
        base = (int(f) * nt + (int(y) // th) * tx + int(x) // tw) * N
        need.update((base + L.astype(np.int64)).tolist())
    print(case, tile, "needed", len(need), "binned", len(got), "plain", len(plain), flush=True)
    assert need <= got, len(need - got)
    assert got <= plain, len(got - plain)
    assert len(got) < len(plain) or case == "c1"


# ------------------------------------------------------------ FP32 forward sanity

def test_gpu_gradients_against_finite_differences_of_the_gpu_forward():
    """Loose sanity check of the GPU's own FP32 forward: central differences
    (steps of ~1e-3 of each parameter) of sum(gC . C) + sum(gD . D) rendered
    on the GPU against the GPU's analytic gradient, for 60 random parameter
    entries whose perturbation flips no discrete decision (list membership,
    clamp, depth hit, branch: the oracle's per-pixel decision signature is
    compared, as the forward is discontinuous there); within 2e-2 of the
    gradient scale of the parameter group."""
    cfg = make_config("c1")
    cam, sc, poses = cfg["cam"], dict(cfg["scene"]), cfg["poses"]
    N = len(sc["pos"])
    mask = np.ones((1, cam["height"], cam["width"]), np.uint8)
    rast = _rast(cam, N, 1)
    gC, gD = random_upstream(mask, seed=31)
    tgC, tgD = torch.as_tensor(gC).cuda(), torch.as_tensor(gD).cuda()
    g = gpu_forward(rast, sc, poses, mask)
    grads = rast.alloc_grads()
    rast.backward_into(g["ws"], g["params"], dev_poses(poses), *g["tensors"][1:], tgC, tgD, grads)
    torch.cuda.synchronize()
    gnp = {k: v.cpu().numpy() for k, v in grads.items()}

    P, recs0, pix, out0 = oracle_forward(cam, sc, poses, mask)

    def loss(scn):
        o = gpu_forward(rast, scn, poses, mask)
        Cc, Dd = o["color"].astype(np.float64), o["depth"].astype(np.float64)
        sig = orc.render(P, orc.project(P, scn, poses), scn, pix)["sig"]
        return float((Cc * gC).sum() + (Dd * gD).sum()), sig

    rng = np.random.default_rng(32)
    checked, worst = 0, 0.0
    fields = [("pos", 3), ("scale", 3), ("rot", 4), ("opacity", 1), ("color", 3)]
    for name, w in fields:
        scale_g = float(np.abs(gnp[name]).max())
        tried = 0
        for i in rng.permutation(N):
            if tried >= 12:
                break
            c = int(rng.integers(w))
            x0 = float(sc[name][i] if w == 1 else sc[name][i, c])
            h = 1e-3 * max(abs(x0), 1e-2)
            vals, idxs = [], []
            for sgn in (1, -1):
                s2 = {k: v.copy() for k, v in sc.items()}
                if w == 1:
                    s2[name][i] = np.float32(x0 + sgn * h)
                else:
                    s2[name][i, c] = np.float32(x0 + sgn * h)
                l, ind = loss(s2)
                vals.append(l)
                idxs.append(ind)
            if not (np.array_equal(idxs[0], out0["sig"]) and np.array_equal(idxs[1], out0["sig"])):
                continue
            hp = float(np.float32(x0 + h)) - float(np.float32(x0 - h))
            fd = (vals[0] - vals[1]) / hp
            an = float(gnp[name][i] if w == 1 else gnp[name][i, c])
            worst = max(worst, abs(fd - an) / max(scale_g, 1e-12))
            tried += 1
            checked += 1
    print("GPU FD sanity: %d entries, worst |fd - grad| / group scale %.2e" % (checked, worst), flush=True)
    assert checked >= 40
    assert worst < 2e-2


# --------------------------------------- Gaussian groups and ranges at their edges

@pytest.mark.parametrize("n,frames", [(1, 1), (15, 2), (17, 1), (64, 3), (129, 2)])
def test_unstable_mask_groups_at_the_edges(n, frames):
    """Groups of Gaussians with a remainder, footprints larger than a block
    of pixels and cut by the image: bit-exact against the oracle."""
    cam = small_cam(61, 43, 60.0)
    rng = np.random.default_rng(n)
    sc = random_scene(rng, n, spread=1.2, smin=0.02, smax=0.3, unstable_frac=0.5)
    sc["unstable"][0] = 1
    poses = np.repeat(identity_pose(), frames, 0)
    poses[:, 9] += 0.1 * np.arange(frames)
    rast = _rast(cam, n, frames)
    m = rast.unstable_mask(dev_params(sc), dev_poses(poses)).cpu().numpy()
    recs = orc.project(orc.make_params(cam), sc, poses)
    assert np.array_equal(m, orc.unstable_mask_image(orc.make_params(cam), recs, sc["unstable"]))


@pytest.mark.parametrize("n", [1, 255, 257, 140_000])
def test_projection_backward_ranges(n):
    """Workgroup ranges of 256 and more Gaussians with few and many of them
    in view: unstable rows in view equal the oracle's chain, unstable rows
    out of view are zero, stable rows are not touched."""
    cam = small_cam(61, 43, 60.0)
    rng = np.random.default_rng(n)
    k = min(n, 300)
    sc = random_scene(rng, n, spread=0.8, unstable_frac=0.5)
    hidden = np.ones(n, bool)
    hidden[rng.permutation(n)[:k]] = False
    sc["pos"][hidden, 2] = -3.0                    # behind the camera
    poses = identity_pose()
    mask = np.ones((1, 43, 61), np.uint8)
    rast = _rast(cam, n, 1)
    params, dp = dev_params(sc), dev_poses(poses)
    C, D, T, I, ws = rast.forward(params, dp, dev_mask(mask))
    gC, gD = random_upstream(mask, seed=3)
    grads = {key: torch.full_like(v, 7.0) for key, v in rast.alloc_grads().items()}
    rast.backward_into(ws, params, dp, D, T, I, torch.as_tensor(gC).cuda(), torch.as_tensor(gD).cuda(), grads)
    torch.cuda.synchronize()
    sub = {key: v[~hidden] for key, v in sc.items()}
    P = orc.make_params(cam)
    recs = orc.project(P, sub, poses)
    pix = orc.masked_pixels(mask)
    f, x, y = pix[:, 0], pix[:, 1], pix[:, 2]
    ref = orc.backward(P, recs, sub, poses, pix, gC[f, y, x], gD[f, y, x])
    un = sc["unstable"] != 0
    for key in ("pos", "scale", "rot", "opacity", "color"):
        g = grads[key].cpu().numpy().reshape(n, -1)
        assert (g[~un] == 7.0).all() and (g[un & hidden] == 0.0).all(), key
        r = np.asarray(ref[key]).reshape(k, -1)[un[~hidden]]
        assert np.linalg.norm(g[un & ~hidden] - r) <= 1e-4 * max(np.linalg.norm(r), 1e-30), key


def _tile_lists(rast, ws, F, nt):
    tend = ws_view(rast, ws, "tile_end", torch.int32, F * nt).cpu().numpy()
    start = ws_view(rast, ws, "tile_start", torch.int32, F * nt).cpu().numpy()
    pairs = ws_view(rast, ws, "pairs", torch.int32, rast.max_pairs).cpu().numpy()
    npx = ws_view(rast, ws, "tile_npx", torch.int32, F * nt).cpu().numpy()
    return [pairs[a:b] for a, b in zip(start, tend)], npx


@pytest.mark.parametrize("n,size,frames,tile,cover,big", [
    (1, (61, 43), 1, (16, 16), 1.0, False), (255, (61, 43), 2, (8, 8), 0.5, False),
    (1025, (130, 70), 1, (16, 16), 1.0, False), (2050, (97, 66), 3, (32, 8), 0.2, False),
    (5000, (128, 96), 1, (16, 16), 0.02, False), (300, (64, 48), 1, (16, 16), 1.0, True),
    (700, (64, 48), 1, (16, 16), 1.0, True), (4096, (33, 17), 1, (16, 16), 1.0, True),
    (4097, (33, 17), 2, (16, 16), 1.0, True), (9000, (33, 17), 1, (16, 16), 1.0, True)])
def test_binning_per_tile_equals_the_general_path(n, size, frames, tile, cover, big):
    """The one-workgroup-per-tile binning of small plans against the general
    path (a plan with sort_cap given): the same lists tile by tile, pixels,
    totals and rendered bits; lists of 0 to 9,000 pairs (rank, LDS, register
    and merge sorts), empty tiles, a second binning with another mask, and a
    capacity that is one pair short."""
    cam = small_cam(*size, 0.9 * size[0])
    rng = np.random.default_rng(n)
    sc = random_scene(rng, n, spread=0.1 if big else 0.9, smin=0.3 if big else 0.01, smax=0.6 if big else 0.08,
                      opaque_frac=0.02 if big else 0.7)
    sc["opacity"] = np.where(sc["opacity"] > 0.5, sc["opacity"], 0.002 if big else sc["opacity"]).astype(np.float32)
    poses = np.repeat(identity_pose(), frames, 0)
    poses[:, 9] += 0.05 * np.arange(frames)
    masks = [(rng.random((frames, size[1], size[0])) < cover).astype(np.uint8) for _ in range(2)]
    masks[0][:, : size[1] // 3] = 0
    nt = -(-size[0] // tile[0]) * -(-size[1] // tile[1])
    got = {}
    for cap in (0, 4096):
        rast = _rast(cam, n, frames, tile_w=tile[0], tile_h=tile[1], sort_cap=cap)
        ws = rast.new_workspace()
        rast.project(ws, *dev_params(sc), dev_poses(poses))
        for k, m in enumerate(masks):
            rast.bin(ws, dev_mask(m))
            out = rast.alloc_outputs()
            rast.render_into(ws, *out)
            st = rast.read_status(ws)
            lists, npx = _tile_lists(rast, ws, frames, nt)
            got[cap, k] = (lists, npx, {key: st[key] for key in ("pairs", "pixels", "items", "overflow", "err", "big_tiles",
                                                                 "restaged_blocks", "status")},
                           [t.cpu().numpy() for t in out])
    for k in range(2):
        a, b = got[0, k], got[4096, k]
        assert a[2] == b[2] and a[2]["status"] == 0
        assert np.array_equal(a[1], b[1])
        for x, y, p in zip(a[0], b[0], a[1]):
            assert np.array_equal(x, y) if p else len(x) == 0
        for x, y in zip(a[3], b[3]):
            assert np.array_equal(x.view(np.uint32), y.view(np.uint32))
    K = got[0, 1][2]["pairs"]
    if K > 1:
        rast = _rast(cam, n, frames, tile_w=tile[0], tile_h=tile[1], max_pairs=K - 1)
        ws = rast.new_workspace()
        rast.project(ws, *dev_params(sc), dev_poses(poses))
        for _ in range(2):
            rast.bin(ws, dev_mask(masks[1]))
            out = rast.alloc_outputs()
            rast.render_into(ws, *out)
            st = rast.read_status(ws)
            assert st["overflow"] == 1 and st["pairs"] == K and st["items"] == 0 and st["status"] != 0
            assert (out[3].cpu().numpy() == -1).all() and not out[0].any()


@pytest.mark.parametrize("n,frames,tile,skew", [(700, 1, (8, 8), False), (3000, 2, (8, 8), False),
                                                (3000, 1, (32, 8), False), (700, 1, (8, 8), True)])
def test_few_ranges_over_many_tiles(n, frames, tile, skew):
    """Binning blocks with tile chunks of about a thousand (few Gaussians,
    thousands of tiles): the oracle's lists.  With most pairs in one block
    (`skew`, and room for four times the pairs over twelve regions) its
    staging region overflows and it enumerates them twice."""
    size = (1142, 767)
    cam = small_cam(*size, 0.8 * size[0])
    sc, poses = _two_pose_scene(1, n=n)
    poses = poses[:frames]
    rng = np.random.default_rng(n)
    mask = (rng.random((frames, size[1], size[0])) < 0.3).astype(np.uint8)
    if skew:
        mask[:, 40:] = 0
        sc["scale"][:256, :2] *= 4.0
        sc["scale"][256:] *= 0.02
    P = orc.make_params(cam, tile=tile)
    recs = orc.project(P, sc, poses)
    pairs = len(orc.bin_pairs(P, recs, mask)["gid"])
    rast = _rast(cam, len(sc["pos"]), frames, tile_w=tile[0], tile_h=tile[1], sort_cap=4096,
                 **({"max_pairs": pairs + 64} if skew else {}))
    g = gpu_forward(rast, sc, poses, mask)
    assert g["status"]["status"] == 0
    assert (g["status"]["restaged_blocks"] > 0) == skew
    _check_pairs(rast, g["ws"], P, recs, mask, frames, len(sc["pos"]), g)


@pytest.mark.parametrize("ipp,share", [(1, 0), (2, 50), (7, 0), (64, 30)])
def test_queue_with_fewer_chunks_than_waves(ipp, share):
    """A queue over a handful of items, from one to less than one chunk per
    wave: every item is taken (the round-robin outputs, bit for bit)."""
    cam = small_cam(100, 75, 90.0)
    sc, poses = _two_pose_scene(11, n=800)
    rng = np.random.default_rng(ipp)
    mask = (rng.random((2, 75, 100)) < 0.4).astype(np.uint8)
    ref = gpu_forward(_rast(cam, 800, 2), sc, poses, mask)
    got = gpu_forward(_rast(cam, 800, 2, items_per_pop=ipp, static_share=share), sc, poses, mask)
    for k in ("color", "depth", "trans", "index"):
        assert np.array_equal(got[k].view(np.uint32), ref[k].view(np.uint32)), k
    assert got["status"]["blend_fwd"] == ref["status"]["blend_fwd"]
    errs = _grad_parity(cam, sc, poses, mask, seed=5, items_per_pop=ipp, static_share=share)
    print("queue gradients", ipp, share, fmt_stats(errs))


@pytest.mark.parametrize("n,frames,size,sh", [(0, 1, (1, 1), 0), (1, 1, (3, 1), 0), (1365, 1, (64, 64), 0),
                                              (1366, 3, (61, 47), 1), (5000, 2, (127, 65), 3)])
def test_cleared_images_and_gradients(n, frames, size, sh):
    """One launch clears all images or gradients: every word, at array sizes
    around a workgroup's 4096, also under a hook on torch's operations (where
    torch's own fills do it) and from a stream of the caller's."""
    from torch.utils._python_dispatch import TorchDispatchMode

    class Seen(TorchDispatchMode):
        def __torch_dispatch__(self, f, types, args=(), kwargs=None):
            return f(*args, **(kwargs or {}))

    from contextlib import nullcontext
    rast = _rast(small_cam(*size, 50.0), n, frames, sh_degree=sh)
    s = torch.cuda.Stream()
    for ctx in (nullcontext(), Seen(), torch.cuda.stream(s)):
        for _ in range(2):   # the second allocation gets memory that was written
            with ctx:
                out = rast.alloc_outputs()
                g = rast.alloc_grads()
                torch.cuda.synchronize()
                assert [tuple(t.shape) for t in out] == [(frames, size[1], size[0], 3)] + 3 * [(frames, size[1], size[0])]
                for t, v in zip(out, (0, -1, 1, -1)):
                    assert bool((t == v).all()) and t.dtype == (torch.int32 if t is out[3] else torch.float32)
                for k, t in g.items():
                    assert t.shape[0] == n and t.dtype == torch.float32 and not bool(t.any()), k
                for t in (*out, *g.values()):
                    t.fill_(7)
                del out, g, t
    assert tuple(rast.alloc_grads("cpu")["rot"].shape) == (n, 4)


@pytest.mark.parametrize("frames,max_pairs", [(19, 0), (20, 0), (19, 1000)])
def test_tile_ranges_over_sixty_four_chunks(frames, max_pairs):
    """19 frames of 143 x 96 tiles are 64 chunks of 4096, 20 are 68 (where one
    workgroup scans the chunks' totals): the oracle's lists and totals; with
    too little room the overflow is reported and nothing is listed."""
    size, n = (1142, 767), 300
    cam = small_cam(*size, 0.8 * size[0])
    sc, poses = _two_pose_scene(1, n=n)
    poses = poses[np.arange(frames) % 2]
    mask = (np.random.default_rng(3).random((frames, size[1], size[0])) < 0.01).astype(np.uint8)
    rast = _rast(cam, n, frames, tile_w=8, tile_h=8, **({"max_pairs": max_pairs} if max_pairs else {}))
    ws = rast.new_workspace()
    rast.project(ws, *dev_params(sc), dev_poses(poses))
    rast.bin(ws, dev_mask(mask))
    st = rast.read_status(ws)
    P = orc.make_params(cam, tile=(8, 8))
    recs = orc.project(P, sc, poses)
    b = orc.bin_pairs(P, recs, mask)
    assert st["pairs"] == len(b["gid"]) and st["pixels"] == int(mask.sum())
    pad = np.zeros((frames, 768, 1144), np.uint8)
    pad[:, :767, :1142] = mask
    if max_pairs:
        assert st["overflow"] == 1 and st["items"] == 0
        assert not ws_view(rast, ws, "tile_end", torch.int32, frames * 143 * 96).any()
        return
    assert st["items"] == int((pad.reshape(frames, 96, 8, 143, 8).sum((2, 4)) > 0).sum())
    _check_pairs(rast, ws, P, recs, mask, frames, n, {"status": st})


def test_sorts_over_more_workgroups_than_a_launch():
    """32 frames of 512 x 512 tiles: the sorts take two launches (8.4M
    workgroups in the first); the last frame's lists are those of a plan of
    one frame, the total 32 times its."""
    need_gpu()
    size, n, F, nt = (4096, 4096), 200, 32, 512 * 512
    cam = small_cam(*size, 0.8 * size[0])
    sc, poses = _two_pose_scene(1, n=n)
    m = torch.zeros((1, size[1], size[0]), dtype=torch.uint8, device="cuda")
    m[:, 3::64, 5::16] = 1
    got = []
    for f in (1, F):
        rast = _rast(cam, n, f, tile_w=8, tile_h=8, sort_cap=4096)
        ws = rast.new_workspace()
        rast.project(ws, *dev_params(sc), dev_poses(poses[np.zeros(f, int)]))
        rast.bin(ws, m.expand(f, -1, -1).contiguous())
        st = rast.read_status(ws)
        end = ws_view(rast, ws, "tile_end", torch.int32, f * nt)[-nt:].cpu().numpy()
        start = ws_view(rast, ws, "tile_start", torch.int32, f * nt)[-nt:].cpu().numpy()
        pairs = ws_view(rast, ws, "pairs", torch.int32, st["pairs"]).cpu().numpy()
        got.append((st["pairs"], st["items"], end - start, pairs[-(st["pairs"] // f):] - (f - 1) * n))
        del ws, rast
    (k1, i1, c1, p1), (kF, iF, cF, pF) = got
    assert k1 > 10000 and kF == F * k1 and iF == F * i1
    assert np.array_equal(c1, cF) and np.array_equal(p1, pF)


@pytest.mark.parametrize("ipp,share,fwd", [(1, 0, -1), (2, 50, 4), (64, 0, 1), (7, 30, 0)])
def test_queue_heads_serve_repeated_launches(ipp, share, fwd):
    """The last pop of a launch clears its queue head: renders and backwards
    repeated on one binning, and after another binning (also an empty one),
    take every item again."""
    cam = small_cam(160, 120, 144.0)
    sc, poses = _two_pose_scene(5, n=900)
    rng = np.random.default_rng(2)
    mask = (rng.random((2, 120, 160)) < 0.5).astype(np.uint8)
    rast = _rast(cam, 900, 2, items_per_pop=ipp, static_share=share, fwd_items_per_pop=fwd)
    prm, ps = dev_params(sc), dev_poses(poses)
    ws = rast.new_workspace()
    rast.project(ws, *prm, ps)
    up = torch.ones((2, 120, 160, 3), device="cuda"), torch.ones((2, 120, 160), device="cuda")
    ref = None
    for k, m in enumerate((mask, mask, np.zeros_like(mask), mask)):
        rast.bin(ws, dev_mask(m))
        for _ in range(2):
            out = rast.alloc_outputs()
            rast.render_into(ws, *out)
            rast.backward_raster(ws, *out[1:], *up)
            st = rast.read_status(ws)
            got = [t.cpu().numpy() for t in out] + [st["blend_fwd"], st["walk_bwd"]]
            if not m.any():
                assert st["items"] == 0 and st["blend_fwd"] == 0 and bool((out[2] == 1).all())
                continue
            ref = ref or got
            for a, b in zip(got, ref):
                assert np.array_equal(a, b), k
    print("queue heads", ipp, share, fwd, ref[-2:])


@pytest.mark.parametrize("n,cover", [(66000, 0.0003), (66000, 0.3), (140000, 0.002)])
def test_collected_rows_give_the_same_pairs(n, cover):
    """Binning ranges of 512 and 768 Gaussians, whose waves collect the
    Gaussians with an active row: few and many of them, some rectangles of
    more than 64 tile rows, and rounds of fewer than 64: the oracle's lists."""
    size = (1142, 767)
    cam = small_cam(*size, 0.8 * size[0])
    sc, poses = _two_pose_scene(1, n=n)
    sc["scale"] *= 0.05
    sc["scale"][::9001, :2] *= 400.0
    rng = np.random.default_rng(4)
    mask = (rng.random((1, size[1], size[0])) < cover).astype(np.uint8)
    rast = _rast(cam, n, 1, tile_w=8, tile_h=8)
    ws = rast.new_workspace()
    rast.project(ws, *dev_params(sc), dev_poses(poses[:1]))
    rast.bin(ws, dev_mask(mask))
    st = rast.read_status(ws)
    assert st["status"] == 0 and st["restaged_blocks"] == 0
    P = orc.make_params(cam, tile=(8, 8))
    recs = orc.project(P, sc, poses[:1])
    _check_pairs(rast, ws, P, recs, mask, 1, n, {"status": st})
    rect = ws_view(rast, ws, "rect", torch.int16, 4 * n).cpu().numpy().reshape(n, 4)[recs["visible"][0] != 0]
    assert ((rect[:, 3] // 8 - rect[:, 2] // 8) >= 64).any()


@pytest.mark.parametrize("n,frames,size,tile", [
    (262_145, 1, (128, 96), 16), (321_587, 1, (128, 96), 16), (393_217, 1, (64, 48), 16), (458_752, 1, (61, 43), 16),
    (567_209, 2, (144, 96), 16), (589_825, 1, (200, 150), 8)])
def test_every_gaussian_of_a_binning_range_is_listed(n, frames, size, tile):
    """Ranges of an odd multiple of 256 Gaussians, halved as often as a small
    image lets them be: the oracle's lists, with the Gaussians in view spread
    over the whole set."""
    cam = small_cam(*size, 0.9 * size[0])
    rng = np.random.default_rng(n)
    sc = random_scene(rng, n, spread=0.8, smin=0.002, smax=0.02, unstable_frac=0.5)
    sc["pos"][rng.random(n) > 0.02, 2] = -3.0      # behind the camera
    poses = np.repeat(identity_pose(), frames, 0)
    poses[:, 9] += 0.05 * np.arange(frames)
    mask = (rng.random((frames, size[1], size[0])) < 0.7).astype(np.uint8)
    rast = _rast(cam, n, frames, tile_w=tile, tile_h=tile, max_pairs=1 << 20)
    ws = rast.new_workspace()
    rast.project(ws, *dev_params(sc), dev_poses(poses))
    rast.bin(ws, dev_mask(mask))
    st = rast.read_status(ws)
    assert st["status"] == 0 and st["pairs"] > 1000
    P = orc.make_params(cam, tile=(tile, tile))
    _check_pairs(rast, ws, P, orc.project(P, sc, poses), mask, frames, n, {"status": st})


@pytest.mark.parametrize("flat,t_eps", [(0.0, 1.5), (0.0, float("inf")), (1e-6, 1.5)])
def test_threshold_above_one_blends_one_gaussian(flat, t_eps):
    """A transmission threshold above 1: a pixel blends the first Gaussian
    of its list that reaches it and stops, whatever that one's opacity; the
    depth and the index still come from the first hit.  Where every opacity
    counts, the outputs are those of the threshold 1, at which any blend ends
    a pixel; with a Gaussian of opacity zero in front of everything, no
    colour is left."""
    cam = small_cam(100, 75, 90.0)
    sc, poses = _two_pose_scene(51, n=3000)
    if flat:
        sc["scale"][:, 2] = flat                   # needle footprints among them
    rng = np.random.default_rng(52)
    mask = (rng.random((2, 75, 100)) < 0.6).astype(np.uint8)
    runs = []
    for e in (1.0, t_eps):
        rast = _rast(cam, 3000, 2, t_eps=e)
        g = gpu_forward(rast, sc, poses, mask)
        gC, gD = random_upstream(mask, seed=53)
        grads = rast.alloc_grads()
        rast.backward_into(g["ws"], g["params"], dev_poses(poses), *g["tensors"][1:], torch.as_tensor(gC).cuda(),
                           torch.as_tensor(gD).cuda(), grads)
        torch.cuda.synchronize()
        runs.append((g, {k: v.cpu().numpy() for k, v in grads.items()}))
    (g0, a), (g1, b) = runs
    assert g1["status"]["blend_fwd"] == g0["status"]["blend_fwd"] > 0
    for k in ("color", "depth", "trans", "index"):
        assert np.array_equal(g0[k].view(np.uint32), g1[k].view(np.uint32)), k
    for k in a:
        assert np.linalg.norm(a[k] - b[k]) <= 1e-5 * np.linalg.norm(a[k]), k
    # an invisible disc over everything, 0.3 m ahead of the first camera
    n = poses[0, :9].reshape(3, 3)[:, 2]
    front = {k: np.concatenate([v[:1], v]) for k, v in sc.items()}
    front["pos"][0], front["scale"][0], front["opacity"][0] = poses[0, 9:] + 0.3 * n, 2.0, 0.0
    g2 = gpu_forward(_rast(cam, 3001, 2, t_eps=t_eps), front, poses, mask)
    ref = gpu_forward(_rast(cam, 3001, 2), front, poses, mask)
    on = mask[0] != 0
    assert not g2["color"][0].any() and (g2["trans"][0] == 1).all()
    assert np.array_equal(g2["index"], ref["index"]) and np.array_equal(g2["depth"], ref["depth"])
    assert (ref["color"][0][on] > 0).any() and g2["status"]["blend_fwd"] >= on.sum()


def _two_sided_tile(k):
    """One 16x16 tile: a Gaussian on the left in front of k on the right,
    none of which reaches the other side."""
    cam = small_cam(16, 16, 20.0)
    x, z = np.full(k + 1, 0.5), 2.0 + 0.01 * np.arange(k + 1)
    x[0] = -0.5
    pos = np.stack([x * z / 2.0, np.full(k + 1, 0.05), z], 1)
    sc = scene_from(pos, np.full((k + 1, 3), 0.05), np.tile([1.0, 0, 0, 0], (k + 1, 1)), np.full(k + 1, 0.05),
                    np.full((k + 1, 3), 0.5))
    return cam, sc


@pytest.mark.parametrize("k", [1, 63, 64, 200])
def test_walk_counter_ends_at_the_last_blend(k):
    """A pixel walks back from the last Gaussian it blended, wherever its
    list ends: one entry for the pixel on the left, all k + 1 for the one on
    the right."""
    cam, sc = _two_sided_tile(k)
    mask = np.zeros((1, 16, 16), np.uint8)
    mask[0, 8, 3] = mask[0, 8, 12] = 1
    rast = _rast(cam, k + 1)
    params, dp = dev_params(sc), dev_poses(identity_pose())
    C, D, T, I, ws = rast.forward(params, dp, dev_mask(mask))
    up = torch.ones_like(C), torch.ones_like(D)
    rast.backward_into(ws, params, dp, D, T, I, *up, rast.alloc_grads())
    st = rast.read_status(ws)
    assert st["pairs"] == k + 1 and st["eval_fwd"] == 2 * (k + 1)
    assert st["blend_fwd"] == st["part_bwd"] == k + 1
    assert st["walk_bwd"] == 1 + (k + 1)


@pytest.mark.parametrize("kw", [{}, dict(items_per_pop=2, static_share=50), dict(depth_mode=1)])
def test_contribution_counter_is_the_last_backwards(kw):
    """A render after the backward, on another binning, moves the blend
    counter and leaves the backward's contributions and walk; a new
    projection clears them."""
    cam = small_cam(100, 75, 90.0)
    sc, poses = _two_pose_scene(61, n=900)
    rng = np.random.default_rng(62)
    masks = [dev_mask((rng.random((2, 75, 100)) < c).astype(np.uint8)) for c in (0.7, 0.2)]
    rast = _rast(cam, 900, 2, **kw)
    params, dp = dev_params(sc), dev_poses(poses)
    C, D, T, I, ws = rast.forward(params, dp, masks[0])
    rast.backward_into(ws, params, dp, D, T, I, torch.ones_like(C), torch.ones_like(D), rast.alloc_grads())
    a = rast.read_status(ws)
    assert a["part_bwd"] == a["blend_fwd"] > 0
    rast.bin(ws, masks[1])
    rast.render_into(ws, C, D, T, I)
    b = rast.read_status(ws)
    assert (b["part_bwd"], b["walk_bwd"]) == (a["part_bwd"], a["walk_bwd"]) and 0 < b["blend_fwd"] < a["blend_fwd"]
    rast.project(ws, *params, dp)
    c = rast.read_status(ws)
    assert c["blend_fwd"] == c["part_bwd"] == c["walk_bwd"] == 0


def test_collected_rows_in_the_widest_tile_chunk():
    """Two frames of 143 x 96 tiles in ranges of 512 Gaussians: enough
    binning blocks that a chunk keeps 12,288 tiles, 69 KB of LDS with the
    collected rows: the oracle's lists."""
    size, n, frames = (1142, 767), 66_000, 2
    cam = small_cam(*size, 0.8 * size[0])
    sc, poses = _two_pose_scene(1, n=n)
    sc["scale"] *= 0.05
    mask = (np.random.default_rng(5).random((frames, size[1], size[0])) < 0.05).astype(np.uint8)
    rast = _rast(cam, n, frames, tile_w=8, tile_h=8, max_pairs=1 << 22)
    ws = rast.new_workspace()
    rast.project(ws, *dev_params(sc), dev_poses(poses))
    rast.bin(ws, dev_mask(mask))
    st = rast.read_status(ws)
    assert st["status"] == 0 and st["restaged_blocks"] == 0
    P = orc.make_params(cam, tile=(8, 8))
    _check_pairs(rast, ws, P, orc.project(P, sc, poses), mask, frames, n, {"status": st})


def _open_strip_scene(n_far=5000, n_near=1800):
    """Opaque surfels in front of all but a strip at the left, and thousands
    of faint Gaussians behind: a few pixels of a pack keep compositing
    through a list that the others have closed."""
    rng = np.random.default_rng(71)
    near = random_scene(rng, n_near, smin=0.03, smax=0.07, opaque_frac=1.0, unstable_frac=0.5)
    z = rng.uniform(0.9, 1.1, n_near)
    near["pos"] = np.stack([rng.uniform(-0.33, 0.6, n_near) * z, rng.uniform(-0.45, 0.45, n_near) * z, z], 1).astype(np.float32)
    far = random_scene(rng, n_far, smin=0.02, smax=0.1, opaque_frac=0.0, unstable_frac=0.5)
    z = rng.uniform(1.5, 3.0, n_far)
    far["pos"] = np.stack([rng.uniform(-0.55, 0.55, n_far) * z, rng.uniform(-0.42, 0.42, n_far) * z, z], 1).astype(np.float32)
    far["opacity"] = rng.uniform(0.005, 0.02, n_far).astype(np.float32)
    return {k: np.concatenate([near[k], far[k]]) for k in near}


@pytest.mark.parametrize("kw", [dict(), dict(tile_w=8, tile_h=8), dict(tile_w=32, tile_h=8),
                                dict(items_per_pop=1, static_share=30)])
def test_culling_follows_the_open_pixels(kw):
    """Packs whose later batches are culled for a few open pixels: image,
    index, depth branch and gradients against the oracle."""
    cam, sc, poses = small_cam(64, 48, 60.0), _open_strip_scene(), identity_pose()
    mask = np.ones((1, 48, 64), np.uint8)
    rast = _rast(cam, len(sc["pos"]), **kw)
    g = gpu_forward(rast, sc, poses, mask)
    P, recs, pix, out = oracle_forward(cam, sc, poses, mask)
    errs = compare_forward(g, pix, out, recs)
    closed = out["trans"].reshape(48, 64) < T_EPS
    assert closed.mean() > 0.2 and (~closed).mean() > 0.1
    few = closed.reshape(6, 8, 8, 8).sum((1, 3))                # closed pixels per 8x8 pack
    assert ((few >= 40) & (few < 64)).any()
    errs.update(_grad_parity(cam, sc, poses, mask, seed=72, **kw))
    print("open strip", kw, fmt_stats(errs))
    assert errs["index_mismatch"] == 0
    assert_parity(errs)


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("depth_mode", [0, 1])
def test_upstream_that_is_no_number_stays_with_the_gaussians_reached(bad, depth_mode):
    """A pack of two pixels with a Gaussian on each and one between them that
    reaches neither: a NaN or an infinity upstream of one pixel leaves the
    gradients of the one between at zero."""
    cam = small_cam(16, 16, 20.0)
    x = np.array([-0.5, 0.0, 0.5])
    sc = scene_from(np.stack([x, np.full(3, 0.05), np.full(3, 2.0)], 1), np.full((3, 3), 0.05),
                    np.tile([1.0, 0, 0, 0], (3, 1)), np.full(3, 0.5), np.full((3, 3), 0.5))
    mask = np.zeros((1, 16, 16), np.uint8)
    mask[0, 8, 3] = mask[0, 8, 12] = 1
    rast = _rast(cam, 3, depth_mode=depth_mode)
    params, dp = dev_params(sc), dev_poses(identity_pose())
    C, D, T, I, ws = rast.forward(params, dp, dev_mask(mask))
    got = []
    for v in (1.0, bad):
        gC, gD = torch.ones_like(C), torch.ones_like(D)
        gC[0, 8, 12], gD[0, 8, 12] = v, v
        g = rast.alloc_grads()
        rast.project(ws, *params, dp)
        rast.bin(ws, dev_mask(mask))
        rast.render_into(ws, C, D, T, I)
        rast.backward_into(ws, params, dp, D, T, I, gC, gD, g)
        got.append({k: t.cpu().numpy() for k, t in g.items()})
    assert rast.read_status(ws)["pairs"] == 3
    for k in got[0]:
        assert not got[0][k][1].any() and not got[1][k][1].any(), k
    assert not np.isfinite(got[1]["color"][2]).any() and np.isfinite(got[0]["color"]).all()
