"""FAST where the per-tile strength lists can go wrong: tiles as full of corners
as suppression allows, blocks whose borders cut mask words, image pitches and
origins that are not multiples of 16 bytes, and images of less than a tile."""
import numpy as np
import pytest

from oracle import fast_oracle as F
from paper_2202_13347_amd import sfoc as S

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def image(kind, H, W, seed):
    rng = np.random.default_rng(seed)
    if kind == "peaks":   # a peak in every second row and column: one corner per 2 x 2 pixels
        img = np.zeros((H, W))
        img[::2, ::2] = 1.0 + rng.random(img[::2, ::2].shape)
    else:
        img = rng.random((H, W))
    return img.astype(np.float32)


@pytest.mark.parametrize("kind", ["peaks", "noise"])
@pytest.mark.parametrize("H,W,pad,off,nby,nbx,per", [(8, 9, 0, 0, 1, 1, 1), (33, 31, 0, 0, 2, 3, 2),
                                                     (96, 128, 0, 0, 1, 1, 32), (97, 131, 1, 0, 13, 17, 1),
                                                     (130, 164, 4, 1, 9, 5, 3), (200, 100, 3, 3, 40, 33, 1)])
def test_lists_match_oracle(kind, H, W, pad, off, nby, nbx, per):
    print("fast lists", kind, H, W, pad, off, nby, nbx, per, flush=True)
    img = image(kind, H, W, H + W)
    buf = torch.zeros(H * (W + pad) + off + 8, device="cuda")
    dev = buf[off:off + H * (W + pad)].view(H, W + pad)[:, :W]
    dev.copy_(torch.from_numpy(img))
    ips, scores, counts = S.detect_ips(dev, 0.0, 0, nby, nbx, per)
    o_ips, o_sc, o_cnt = F.detect(img, 0.0, 0, nby, nbx, per)
    assert np.array_equal(counts.reshape(-1), np.asarray(o_cnt).reshape(-1))
    assert np.array_equal(ips.cpu().numpy(), o_ips) and np.array_equal(scores, o_sc)   # exact, no rounding involved
