"""GPU parity of frame-to-model tracking (Sec. 3.2, Eq. 10) against
oracle/icp.py, through the C ABI: the rendered normal map (bit-exact), the
data association and normal equations of every ICP iteration given the
pose the GPU used (pair counts exact, sums within binary64 summation
order), recovery of a known motion, and tracking on the rasterizer's own
depth and normal renders."""
import numpy as np
import pytest
import torch

from oracle import icp as oicp
from oracle import oracle as orc
from tests.gpu_helpers import dev_poses, gpu_forward, need_gpu
from tests.scenes_small import random_pose, random_scene, small_cam
from tests.test_oracle_icp import corner_maps

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()
    from paper_2404_19706_amd import lib
    lib()
    yield


def _t(a, dt=None):
    t = torch.as_tensor(np.ascontiguousarray(a)).cuda()
    return t if dt is None else t.to(dt)


def test_normal_map_is_bit_exact():
    from paper_2404_19706_amd import Rasterizer
    cam = small_cam(100, 75, 90.0)
    rng = np.random.default_rng(100)
    pose_a, Rg, tg = random_pose(rng)
    target = tg + 2.0 * Rg[:, 2]
    from rtg_synth import look_at
    poses = np.stack([pose_a, look_at(tg + 0.3 * Rg[:, 0], target, up=-Rg[:, 1])])
    sc = random_scene(rng, 1500, centre=target, spread=0.6)
    mask = (rng.random((2, 75, 100)) < 0.6).astype(np.uint8)
    rast = Rasterizer(cam, 1500, 2)
    g = gpu_forward(rast, sc, poses, mask)
    normals = torch.full((2, 75, 100, 3), 7.0, device="cuda")
    rast.render_normals_into(g["ws"], normals)
    torch.cuda.synchronize()
    P = orc.make_params(cam)
    recs = orc.project(P, sc, poses)
    pix = orc.masked_pixels(mask)
    out = orc.render(P, recs, sc, pix)
    ref = oicp.normal_map(P, recs, out, pix, 75, 100)
    got = normals.cpu().numpy()
    f, x, y = pix[:, 0], pix[:, 1], pix[:, 2]
    assert np.array_equal(got[f, y, x], ref[f, y, x].astype(np.float32))
    assert (got[mask == 0] == 7.0).all()                     # unrendered pixels untouched
    assert (out["index"] >= 0).sum() > 1000


def _motion(pose_m, xi):
    dR, dt = oicp.se3_exp(np.asarray(xi))
    R0, t0 = pose_m[:9].reshape(3, 3), pose_m[9:]
    return np.concatenate([(dR @ R0).ravel(), dR @ t0 + dt])


def test_icp_iterations_match_oracle_and_recover_the_motion():
    from paper_2404_19706_amd import tracking
    cam = small_cam(320, 240, 280.0)
    pose_m = np.concatenate([np.eye(3).ravel(), [0.1, 0.2, 0.0]])
    pose_true = _motion(pose_m, [0.01, -0.008, 0.006, 0.015, -0.01, 0.012])
    Dm, Nm = corner_maps(cam, pose_m)
    Din, _ = corner_maps(cam, pose_true)
    prm = tracking.icp_params()
    pose, trace = tracking.icp(cam, _t(Din), _t(Dm), _t(Nm), _t(pose_m), _t(pose_m), prm, trace=True)
    torch.cuda.synchronize()
    pose, trace = pose.cpu().numpy(), trace.cpu().numpy()
    assert np.abs(pose - pose_true).max() < 1e-5, np.abs(pose - pose_true).max()
    T_ref, tr_ref = oicp.icp(cam, Din, Dm, Nm, pose_m, pose_m, iters=(10, 5, 4))
    assert np.abs(pose - T_ref).max() < 1e-9
    # every iteration, from the pose the GPU used
    lv = oicp.levels_of(cam, Din, Dm, Nm, 3)
    row = 0
    for l, n_it in ((2, 4), (1, 5), (0, 10)):
        lin, lmo, K = lv[l]
        for _ in range(n_it):
            T = trace[row, :12]
            ok, p, q, n = oicp.associate(lin, lmo, K, T, pose_m, 0.1, 0.3420201433256687)
            A, b, err, cnt = oicp.normal_equations(ok, p, q, n)
            assert int(trace[row, 13]) == cnt, (row, trace[row, 13], cnt)
            iu = np.triu_indices(6)
            np.testing.assert_allclose(trace[row, 14:35], A[iu], rtol=1e-10, atol=1e-9 * np.abs(A).max())
            np.testing.assert_allclose(trace[row, 35:41], b, rtol=1e-9, atol=1e-9 * np.abs(b).max() + 1e-12)
            assert trace[row, 12] == pytest.approx(err, rel=1e-9, abs=1e-15)
            row += 1
    assert trace[0, 13] > 1000


def test_tracking_on_rendered_depth_and_normals():
    """The model rendered by the rasterizer (depth by Eq. 5 and the normal
    map) at one pose, the input frame's depth rendered at a pose moved by a
    small motion: ICP from the model pose lands near the true pose."""
    from paper_2404_19706_amd import Rasterizer, tracking
    from rtg_synth import make_config
    cfg = make_config("c2")
    cam, sc, poses = cfg["cam"], cfg["scene"], cfg["poses"]
    N = len(sc["pos"])
    pose_m = np.asarray(poses[0], np.float64)
    pose_true = _motion(pose_m, [0.004, -0.003, 0.002, 0.01, -0.006, 0.008])
    rast = Rasterizer(cam, N, 2)
    mask = np.ones((2, cam["height"], cam["width"]), np.uint8)
    g = gpu_forward(rast, sc, np.stack([pose_m, pose_true]), mask)
    normals = torch.zeros((2, cam["height"], cam["width"], 3), device="cuda")
    rast.render_normals_into(g["ws"], normals)
    D = g["tensors"][1]
    pose = tracking.icp(cam, D[1].contiguous(), D[0].contiguous(), normals[0].contiguous(), _t(pose_m),
                        _t(pose_m))
    torch.cuda.synchronize()
    err0 = np.abs(pose_m - pose_true).max()
    err = np.abs(pose.cpu().numpy() - pose_true).max()
    print("tracking error %.2e (start %.2e)" % (err, err0))
    assert err < 0.1 * err0


@pytest.mark.parametrize("w,h,levels", [(2, 2, 1), (16, 16, 1), (65, 7, 1), (45, 23, 2), (64, 40, 3), (131, 97, 3),
                                        (130, 66, 2), (517, 389, 3)])
def test_icp_pass_edges(w, h, levels):
    """Strips, rows and partial-row places at their edges: a single
    workgroup (images of a few hundred pixels), widths one off a strip of 64
    columns, odd sizes in the pyramid, and too few pairs for an update; every
    iteration's sums from the pose it used, as above."""
    from paper_2404_19706_amd import tracking
    cam = small_cam(w, h, 0.9 * w)
    pose_m = np.concatenate([np.eye(3).ravel(), [0.1, 0.2, 0.0]])
    Dm, Nm = corner_maps(cam, pose_m)
    Din, _ = corner_maps(cam, _motion(pose_m, [0.004, -0.003, 0.002, 0.006, -0.005, 0.004]))
    iters = (3, 2, 2)
    start = _t(pose_m)
    pose, trace = tracking.icp(cam, _t(Din), _t(Dm), _t(Nm), _t(pose_m), start, tracking.icp_params(levels, iters),
                               trace=True)
    torch.cuda.synchronize()
    trace = trace.cpu().numpy()
    assert np.array_equal(start.cpu().numpy(), pose_m)
    lv = oicp.levels_of(cam, Din, Dm, Nm, levels)
    row = 0
    for l in range(levels - 1, -1, -1):
        lin, lmo, K = lv[l]
        for _ in range(iters[l]):
            T = trace[row, :12]
            ok, p, q, n = oicp.associate(lin, lmo, K, T, pose_m, 0.1, 0.3420201433256687)
            A, b, err, cnt = oicp.normal_equations(ok, p, q, n)
            assert int(trace[row, 13]) == cnt, (row, trace[row, 13], cnt)
            iu = np.triu_indices(6)
            np.testing.assert_allclose(trace[row, 14:35], A[iu], rtol=1e-10, atol=1e-9 * np.abs(A).max())
            np.testing.assert_allclose(trace[row, 35:41], b, rtol=1e-9, atol=1e-9 * np.abs(b).max() + 1e-12)
            assert not trace[row, 41:].any()
            row += 1
    assert row == len(trace) and np.isfinite(pose.cpu().numpy()).all()


def _plane_maps(cam, pose, planes):
    """Depth and camera-frame normals of the nearest plane n . x = d."""
    R, t = pose[:9].reshape(3, 3), pose[9:]
    y, x = np.mgrid[: cam["height"], : cam["width"]] + 0.5
    ray = np.stack([(x - cam["cx"]) / cam["fx"], (y - cam["cy"]) / cam["fy"], np.ones_like(x)], -1)
    D, N = np.full(x.shape, np.inf), np.zeros(ray.shape)
    for n, d in planes:
        nc = np.asarray(n, np.float64) @ R
        with np.errstate(divide="ignore"):
            z = (d - np.dot(n, t)) / (ray @ nc)
        near = (z > 0) & (z < D)
        D[near], N[near] = z[near], nc
    N[(N * ray).sum(-1) > 0] *= -1
    return np.where(np.isfinite(D), D, 0).astype(np.float32), N.astype(np.float32)


def _halves(v):
    """The sum over the last axis (64 lanes), lane l and l ^ 32 first."""
    while v.shape[-1] > 1:
        o = v.shape[-1] // 2
        v = v[..., :o] + v[..., o:]
    return v[..., 0]


def _ordered_sums(ok, p, q, n):
    """The 29 terms of the normal equations in the library's order: pixel i
    to thread i % 256 of block (i // 256) % B, whose sums run in pixel order;
    then lanes, waves and blocks in their fixed tree."""
    r = oicp._dot(p - q, n)
    J = np.concatenate([oicp._cross(p, n), n], -1)
    cols = [J[..., i] * J[..., j] for i in range(6) for j in range(i, 6)]
    cols += [J[..., i] * r for i in range(6)] + [r * r, np.ones_like(r)]
    px = ok.size
    B = min(-(-px // 256), 512)
    rounds = -(-px // (256 * B))
    t = np.zeros((29, rounds * B * 256))
    t[:, :px] = [np.where(ok, c, 0.0).ravel() for c in cols]
    s = np.zeros((29, B, 4, 64))
    for k in range(rounds):
        s = s + t.reshape(29, rounds, B, 4, 64)[:, k]
    w = _halves(s)
    rows = np.zeros((29, 512))
    rows[:, :B] = (w[..., 0] + w[..., 1]) + (w[..., 2] + w[..., 3])
    w = _halves((rows[:, :256] + rows[:, 256:]).reshape(29, 4, 64))
    return (w[:, 0] + w[:, 1]) + (w[:, 2] + w[:, 3])


def _ordered_solve(tot):
    """xi of the Cholesky solve in its fixed order, or None (no update)."""
    A = np.zeros((6, 6))
    A[np.triu_indices(6)] = tot[:21]
    L = np.zeros((6, 6))
    if tot[28] < 6:
        return None
    for i in range(6):
        for j in range(i + 1):
            acc = A[j, i]
            for m in range(j):
                acc = acc - L[i, m] * L[j, m]
            if i == j and not acc > 0.0:
                return None
            L[i, j] = np.sqrt(acc) if i == j else acc / L[j, j]
    y, xi = np.zeros(6), np.zeros(6)
    for i in range(6):
        acc = tot[21 + i]
        for m in range(i):
            acc = acc - L[i, m] * y[m]
        y[i] = acc / L[i, i]
    for i in range(5, -1, -1):
        acc = y[i]
        for m in range(i + 1, 6):
            acc = acc - L[m, i] * xi[m]
        xi[i] = acc / L[i, i]
    return -xi


@pytest.mark.parametrize("w,h,levels", [(33, 17, 1), (97, 66, 3), (131, 97, 2), (640, 400, 2)])
@pytest.mark.parametrize("view", ["wall", "slanted", "two planes", "corner"])
def test_views_that_do_not_fix_the_pose(view, w, h, levels):
    """Where fewer than three independent normals are in view, the last
    pivots of the 6x6 system are rounding noise, and whether the pose moves,
    and where to, follows the order of every sum: the trace holds the sums of
    the stated order bit for bit, and each pose is the one before it, bit for
    bit, where that order refuses a pivot, else exp(xi) of it.  Tolerance of
    the latter: a library's sin and cos within a unit in the last place each,
    through 1 - cos over th^2, a dozen roundings beside."""
    from paper_2404_19706_amd import tracking
    cam = small_cam(w, h, 0.9 * w)
    pose_m = np.concatenate([np.eye(3).ravel(), [0.1, 0.2, 0.0]])
    planes = {"wall": [((0, 0, 1), 2.0)], "slanted": [((0.3, -0.2, 1.0), 2.0)],
              "two planes": [((0, 0, 1), 2.0), ((0, 1, 0.2), 0.9)],
              "corner": [((0, 0, 1), 2.0), ((0, 1, 0.2), 0.7), ((1, 0, 0.3), 0.8)]}[view]
    rng = np.random.default_rng(w)
    Dm, Nm = _plane_maps(cam, pose_m, planes)
    Din, _ = _plane_maps(cam, _motion(pose_m, [0.004, -0.003, 0.002, 0.006, -0.005, 0.004]), planes)
    Din = Din * (1 + 0.002 * rng.standard_normal(Din.shape)) * (rng.random(Din.shape) > 0.03)
    Din = Din.astype(np.float32)
    iters = (4, 3, 2)
    pose, trace = tracking.icp(cam, _t(Din), _t(Dm), _t(Nm), _t(pose_m), _t(pose_m),
                               tracking.icp_params(levels, iters), trace=True)
    torch.cuda.synchronize()
    pose, trace = pose.cpu().numpy(), trace.cpu().numpy()
    lv = oicp.levels_of(cam, Din, Dm, Nm, levels)
    eps = np.finfo(np.float64).eps
    row, moved = 0, 0
    for l in range(levels - 1, -1, -1):
        lin, lmo, K = lv[l]
        for _ in range(iters[l]):
            T = trace[row, :12]
            with np.errstate(all="ignore"):
                tot = _ordered_sums(*oicp.associate(lin, lmo, K, T, pose_m, 0.1, 0.3420201433256687))
                xi = _ordered_solve(tot)
            assert np.array_equal(trace[row, 14:41], tot[:27]) and np.array_equal(trace[row, 12:14], tot[27:]), row
            row += 1
            got = trace[row, :12] if row < len(trace) else pose
            if xi is None:
                assert np.array_equal(got, T), row
                continue
            moved += 1
            th = np.sqrt((xi[0] * xi[0] + xi[1] * xi[1]) + xi[2] * xi[2])
            W = np.array([[0, -xi[2], xi[1]], [xi[2], 0, -xi[0]], [-xi[1], xi[0], 0]])
            a, b, c = np.sin(th) / th, (1 - np.cos(th)) / (th * th), (th - np.sin(th)) / (th * th * th)
            R, V = np.eye(3) + a * W + b * (W @ W), np.eye(3) + b * W + c * (W @ W)
            R0, t0 = T[:9].reshape(3, 3), T[9:]
            ref = np.concatenate([(R @ R0).ravel(), R @ t0 + V @ xi[3:]])
            lim = 32 * eps * (1 + np.abs(T[9:]).max() + np.abs(xi[3:]).max() * (1 + 1 / th))
            assert np.abs(got - ref).max() <= lim, (row, np.abs(got - ref).max(), lim)
    print(view, (w, h), "updates", moved, "of", row, "moved %.3g" % np.abs(pose - pose_m).max())
    assert row == len(trace)
