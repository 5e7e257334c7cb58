"""The K = 1, rates 1-3 describe kernel over filter banks that take each of its
paths: every radius 1 to 12 and beyond, sigmas of the first order, of the
second and of both, one to sixteen orientations (an odd number among them),
each rectification, tiles at the image border, ragged and alone."""
import numpy as np
import pytest

from oracle import sfoc_oracle as O
from paper_2202_13347_amd import sfoc as S
from paper_2202_13347_amd import synth

from tests.gpu_util import DESC_TOL, desc_condition, to_chw
from tests.test_gpu_parity import dev, oparams

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def sig(*radii):
    return tuple((r - 0.2) / 3.0 for r in radii)   # radius ceil(3 sigma)


# The tolerance of the other describe tests (DESC_TOL times the pixel's
# condition): the sums here have as many terms as theirs, up to 3 x 29.
@pytest.mark.parametrize("shape,n,r1,r2,rect", [
    ((33, 64), 1, (1,), (2,), 0),
    ((45, 70), 2, (4,), (5,), 1),
    ((64, 31), 3, (6, 7), (7,), 2),
    ((70, 40), 4, (13,), (13, 14), 0),
    ((40, 97), 6, (8, 9), (3,), 0),
    ((35, 35), 12, (2, 10), (10, 1), 0),
    ((66, 34), 16, (11,), (12, 3), 0),
])
def test_filter_banks(shape, n, r1, r2, rect):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print("describe", shape, n, r1, r2, rect, flush=True)
    img = synth.make_pair(17, shape, 2.0).ref
    p = S.params(n_orient=n, s1=sig(*r1), s2=sig(*r2), rectify=rect)
    desc, i1, i2 = S.describe(dev(img), p)
    torch.cuda.synchronize()
    F = O.sfoc(img.astype(np.float64), oparams(p))
    g = desc.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(g - to_chw(F)) <= DESC_TOL * desc_condition(img, oparams(p)))
    own1, own2 = O.integral_feature_images(g.transpose(1, 2, 0))
    assert np.abs(i1.cpu().numpy() - own1).max() <= 1e-9 * max(1.0, np.abs(own1).max())
    assert np.abs(i2.cpu().numpy() - own2).max() <= 1e-9 * max(1.0, np.abs(own2).max())
