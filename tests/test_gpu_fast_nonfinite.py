"""FAST on images with pixels that are not finite (outside what the header
promises, but callers have nodata areas): a difference that is NaN counts neither
for nor against an arc, and such a pixel is no corner."""
import numpy as np
import pytest

from oracle import fast_oracle as F
from paper_2202_13347_amd import sfoc as S

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def strength(img, b):
    a = np.asarray(img, np.float32)
    H, W = a.shape
    V = np.full((H, W), -np.inf, np.float32)
    c = a[b:H - b, b:W - b]
    with np.errstate(invalid="ignore"):
        u = np.stack([a[b + dy:H - b + dy, b + dx:W - b + dx] for dy, dx in F.CIRCLE]) - c[None]
        best = np.full(c.shape, -np.inf, np.float32)
        for k in range(16):
            arc = u[[(k + j) % 16 for j in range(F.ARC)]]
            best = np.fmax(best, np.fmax(np.fmin.reduce(arc, 0), -np.fmax.reduce(arc, 0)))
    V[b:H - b, b:W - b] = best
    return V


def image(kind, H, W):
    rng = np.random.default_rng(H)
    img = rng.random((H, W)).astype(np.float32)
    img[1::5, ::4] += 2
    if kind == "area":            # nodata above a slanted border
        y, x = np.mgrid[:H, :W]
        img[y < 20 + x // 3] = np.nan
    elif kind == "rows":          # every third row
        img[::3] = np.nan
    else:
        bad = rng.random((H, W)) < 0.03
        img[bad] = rng.choice(np.array([np.nan, np.inf, -np.inf], np.float32), int(bad.sum()))
    return img


@pytest.mark.parametrize("kind", ["area", "rows", "scattered"])
@pytest.mark.parametrize("H,W,pad,nby,nbx,per", [(96, 128, 0, 3, 4, 32), (97, 131, 1, 13, 17, 1), (33, 40, 0, 1, 1, 32)])
def test_nan_and_inf(kind, H, W, pad, nby, nbx, per, monkeypatch):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print("fast nonfinite", kind, H, W, flush=True)
    img = image(kind, H, W)
    dev = torch.zeros(H, W + pad, device="cuda")[:, :W]
    dev.copy_(torch.from_numpy(img))
    ips, scores, counts = S.detect_ips(dev, 0.05, 0, nby, nbx, per)
    monkeypatch.setattr(F, "strength", strength)
    o_ips, o_sc, o_cnt = F.detect(img, 0.05, 0, nby, nbx, per)
    assert len(o_ips) > 10 or kind == "area"
    np.testing.assert_array_equal(counts.reshape(-1), np.asarray(o_cnt).reshape(-1))
    np.testing.assert_array_equal(ips.cpu().numpy(), o_ips)
    np.testing.assert_array_equal(scores, o_sc)
