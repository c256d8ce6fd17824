"""GPU parity of the mapping-iteration steps around the backward (Sec. 3.2,
Eq. 8-9; "Keyframes and global optimization") against oracle/optim.py,
through the C ABI: the transparent L2 regulariser (loss and gradient rows),
the confidence-weighted fusion (bit-exact, RGB and SH rows) and the
top colour-error pixel selection (bit-exact masks, with ties)."""
import numpy as np
import pytest
import torch

from oracle import optim
from tests.gpu_helpers import need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()
    from paper_2404_19706_amd import lib
    lib()
    yield


def _t(a):
    return torch.as_tensor(np.ascontiguousarray(a)).cuda()


def test_reg_l2_matches_oracle():
    from paper_2404_19706_amd import mapping
    rng = np.random.default_rng(0)
    n = 5000
    init = {"pos": rng.standard_normal((n, 3)).astype(np.float32),
            "scale": rng.uniform(0.001, 0.01, (n, 3)).astype(np.float32),
            "rot": rng.standard_normal((n, 4)).astype(np.float32)}
    cur = {k: (v + 1e-3 * rng.standard_normal(v.shape)).astype(np.float32) for k, v in init.items()}
    tr = (rng.random(n) < 0.3).astype(np.uint8)
    un = (rng.random(n) < 0.6).astype(np.uint8)
    g0 = {k: rng.standard_normal(v.shape).astype(np.float32) for k, v in init.items()}
    grads = {k: _t(v) for k, v in g0.items()}
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    mapping.reg_l2(1000.0, _t(tr), _t(un), {k: _t(v) for k, v in cur.items()}, {k: _t(v) for k, v in init.items()},
                   grads, loss)
    torch.cuda.synchronize()
    ref_loss, ref_g = optim.reg_l2(1000.0, tr, un, cur, init)
    assert abs(loss.item() - ref_loss) <= 1e-12 * ref_loss
    for k in ("pos", "scale", "rot"):
        got = grads[k].cpu().numpy().astype(np.float64)
        exp = g0[k].astype(np.float64) + ref_g[k]
        np.testing.assert_allclose(got, exp, rtol=1e-6, atol=1e-6)
        # rows that are not unstable-and-transparent are untouched, bit for bit
        other = (tr == 0) | (un == 0)
        assert np.array_equal(grads[k].cpu().numpy()[other], g0[k][other])


@pytest.mark.parametrize("width", [3, 48])
def test_fuse_is_bit_exact(width):
    from paper_2404_19706_amd import mapping
    rng = np.random.default_rng(1 + width)
    n = 3000
    shapes = {"pos": (n, 3), "scale": (n, 3), "rot": (n, 4),
              "color": (n, 3) if width == 3 else (n, width // 3, 3)}
    prev = {k: rng.standard_normal(s).astype(np.float32) for k, s in shapes.items()}
    cur = {k: rng.standard_normal(s).astype(np.float32) for k, s in shapes.items()}
    eta_prev = rng.integers(0, 300, n).astype(np.int32)
    eta_cur = (eta_prev + rng.integers(0, 60, n)).astype(np.int32)
    eta_prev[:10] = 0
    eta_cur[:5] = 0                                  # eta' = 0 rows
    dcur = {k: _t(v) for k, v in cur.items()}
    mapping.fuse(_t(eta_prev), _t(eta_cur), {k: _t(v) for k, v in prev.items()}, dcur)
    torch.cuda.synchronize()
    ref = optim.fuse(eta_prev, eta_cur, prev, cur)
    for k in shapes:
        assert np.array_equal(dcur[k].cpu().numpy().view(np.uint32), ref[k].view(np.uint32)), k


@pytest.mark.parametrize("frac", [0.0, 0.4, 0.9, 1.0])
def test_top_error_selection_is_bit_exact(frac):
    from paper_2404_19706_amd import mapping
    rng = np.random.default_rng(int(frac * 10) + 7)
    F, H, W = 3, 240, 320
    Cin = rng.random((F, H, W, 3)).astype(np.float32)
    Cr = (Cin + 0.2 * rng.standard_normal((F, H, W, 3))).astype(np.float32)
    Cr[0, :60] = Cin[0, :60]                       # a quarter of frame 0 with zero error (ties)
    Cr[1, :, :100] = np.round(Cr[1, :, :100] * 8) / 8   # coarse values: many equal errors
    Cin[1, :, :100] = np.round(Cin[1, :, :100] * 8) / 8
    m = mapping.select_top_error(_t(Cr), _t(Cin), frac)
    torch.cuda.synchronize()
    ref = optim.select_top_error(Cr, Cin, frac)
    assert np.array_equal(m.cpu().numpy(), ref)
    k = int(np.floor(frac * H * W))
    for f in range(F):
        assert ref[f].sum() >= k


@pytest.mark.parametrize("frames,h,w,offset", [(1, 1, 1, 0), (2, 1, 3, 0), (3, 2, 2, 0), (2, 37, 53, 0), (2, 64, 60, 0),
                                               (2, 64, 60, 1), (5, 130, 126, 0), (1, 300, 301, 0)])
def test_top_error_selection_at_the_edges(frames, h, w, offset):
    """Frames of a few pixels, frame sizes that are and are not multiples of
    four, images that start off 16-byte alignment (one float in), errors that
    share their leading digits or are all alike: the oracle's masks."""
    from paper_2404_19706_amd import mapping
    rng = np.random.default_rng(7)
    for spread in (0.0, 1e-6, 1.0):
        Cin = rng.random((frames, h, w, 3)).astype(np.float32)
        Cr = (Cin + spread * rng.standard_normal(Cin.shape)).astype(np.float32)

        def t(a):
            buf = torch.zeros(a.size + offset, device="cuda")
            buf[offset:] = torch.as_tensor(a.ravel())
            return buf[offset:].view(a.shape)
        for frac in (0.0, 0.4, 1.0):
            m = mapping.select_top_error(t(Cr), t(Cin), frac)
            torch.cuda.synchronize()
            assert np.array_equal(m.cpu().numpy(), optim.select_top_error(Cr, Cin, frac)), (spread, frac)


@pytest.mark.parametrize("n,width,offset", [(1, 3, 0), (255, 5, 0), (256, 12, 0), (257, 27, 0), (511, 48, 0), (300, 1, 0),
                                            (257, 3, 1), (300, 48, 1)])
def test_fuse_at_the_edges(n, width, offset):
    """Workgroups of 256 rows and their remainders, every kind of row width,
    and arrays off 16-byte alignment: bit-exact against the oracle."""
    from paper_2404_19706_amd import mapping
    rng = np.random.default_rng(width + n)

    def t(a):
        buf = torch.zeros(a.size + offset, dtype=torch.float32, device="cuda")
        buf[offset:] = torch.as_tensor(a.ravel())
        return buf[offset:].view(a.shape)
    shapes = {"pos": (n, 3), "scale": (n, 3), "rot": (n, 4), "color": (n, width)}
    prev = {k: rng.standard_normal(s).astype(np.float32) for k, s in shapes.items()}
    cur = {k: rng.standard_normal(s).astype(np.float32) for k, s in shapes.items()}
    eta_prev = rng.integers(0, 300, n).astype(np.int32)
    eta_cur = (eta_prev + rng.integers(0, 60, n)).astype(np.int32)
    eta_prev[n // 2], eta_cur[n // 2] = 0, 0
    dcur = {k: t(v) for k, v in cur.items()}
    mapping.fuse(_t(eta_prev), _t(eta_cur), {k: t(v) for k, v in prev.items()}, dcur)
    torch.cuda.synchronize()
    ref = optim.fuse(eta_prev, eta_cur, prev, cur)
    for k in shapes:
        assert np.array_equal(dcur[k].cpu().numpy().view(np.uint32), ref[k].view(np.uint32)), k


@pytest.mark.parametrize("n,deg,frac", [(1, 0, 1.0), (255, 3, 0.3), (256, 1, 1.0), (257, 2, 0.05), (700, 0, 0.0)])
def test_adam_by_elements_at_the_edges(n, deg, frac):
    """Every parameter group at workgroup remainders, with all, few and no
    unstable rows, against the oracle's Adam (tolerances of the tests of
    whole optimisation steps); stable rows keep their bits."""
    from oracle import oracle as orc
    from paper_2404_19706_amd import Rasterizer
    from tests.scenes_small import small_cam
    rng = np.random.default_rng(n + deg)
    K = (deg + 1) ** 2
    rast = Rasterizer(small_cam(40, 30, 40.0), n, 1, max_pairs=1 << 10, sh_degree=deg)
    shapes = {"pos": (n, 3), "scale": (n, 3), "rot": (n, 4), "color": rast.color_shape}
    p0 = {k: rng.standard_normal(s).astype(np.float32) for k, s in shapes.items()}
    p0["scale"] = np.exp(0.3 * p0["scale"]).astype(np.float32)
    g = {k: rng.standard_normal(s).astype(np.float32) for k, s in shapes.items()}
    un = (rng.random(n) < frac).astype(np.uint8)
    d = {k: _t(v) for k, v in p0.items()}
    m, v, step = rast.alloc_adam_state()
    lr = (1e-3, 2e-3, 1.5e-3, 5e-4, 2.5e-5)
    params = (d["pos"], d["scale"], d["rot"], torch.ones(n, device="cuda"), d["color"], _t(un))
    rast.adam(params, {k: _t(x) for k, x in g.items()}, m, v, step, lr=lr, eps=1e-15)
    torch.cuda.synchronize()
    rate = {"pos": lr[0], "rot": lr[2]}
    col0, gc = p0["color"].reshape(n, 3 * K), g["color"].reshape(n, 3 * K)
    z = lambda a: (np.zeros(a.shape), np.zeros(a.shape))   # noqa: E731
    exp = {k: orc.adam_step(p0[k], g[k], *z(p0[k]), 1, rate[k], un, eps=1e-15)[0] for k in rate}
    exp["scale"] = np.exp(orc.adam_step(np.log(p0["scale"].astype(np.float64)), p0["scale"] * g["scale"],
                                        *z(p0["scale"]), 1, lr[1], un, eps=1e-15)[0])
    exp["color"] = np.concatenate([orc.adam_step(col0[:, a:b], gc[:, a:b], *z(col0[:, a:b]), 1, r, un, eps=1e-15)[0]
                                   for a, b, r in ((0, 3, lr[3]), (3, 3 * K, lr[4]))], 1)
    for k in shapes:
        got = d[k].cpu().numpy().reshape(n, -1)
        assert np.allclose(got, exp[k], rtol=1e-5, atol=1e-6), k
        assert np.array_equal(got[un == 0], p0[k].reshape(n, -1)[un == 0]), k
    assert not m.cpu().numpy()[un == 0].any() and int(step.item()) == 1
