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
