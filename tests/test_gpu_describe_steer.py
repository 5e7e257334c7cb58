"""Steering in the general describe kernel bit for bit.  With K = 0 nothing is
smoothed, and with eps = 1 and responses below 2^-13 the norm is 1: a channel is its
steered response.  Channel 0 is then a basis response itself, as is the channel at
90 degrees, and every other channel of the order one fused multiply-add of theirs."""
import math

import numpy as np
import pytest

from paper_2202_13347_amd import sfoc as S

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def fma32(a, b, c):
    """float32 fused multiply-add (the float64 sum rounded to odd)."""
    p, c = np.float64(a) * b.astype(np.float64), c.astype(np.float64)
    s = p + c
    t = s - p
    err = (p - (s - t)) + (c - t)
    even = (s.view(np.int64) & 1) == 0
    return np.where((err != 0) & even, np.nextafter(s, np.copysign(np.inf, err)), s).astype(np.float32)


# (an image that is constant along y: the mixed second derivative is exactly zero)
@pytest.mark.parametrize("orient,second", [(2, False), (4, False), (6, False), (8, False), (2, True), (4, True),
                                           (6, True), (8, True), (12, True), (16, True)])
def test_steered_responses(orient, second):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print("steer", orient, second, flush=True)
    rng = np.random.default_rng(orient)
    img = 1e-5 * rng.random((70, 66))
    if second:
        img[:] = 1e-5 * np.cumsum(rng.random(66) - 0.5)
    p = S.params(n_orient=orient, s1=(1.0, 2.0), s2=(1.5,), K=0, dil=(1,), eps=1.0, rectify="signed",
                 second_order=second)
    d = S.describe(torch.from_numpy(img.astype(np.float32)).cuda(), p, integrals=False)[0].cpu().numpy()
    assert np.abs(d).max() < 2.0 ** -14 and len(np.unique(d)) > 1000 / (1 + 10 * second)
    f32 = np.float32
    for order in (0, 1)[second:1 + second]:
        b0, b1 = d[order * orient], d[order * orient + orient // 2]
        # (the cosine of 90 degrees is 6e-17: b1 is the response itself where it is not far below b0)
        sure = np.abs(b1) > 1e-6 * np.abs(b0)
        assert sure.mean() > 0.5
        for k in range(orient):
            cs, sn = math.cos(k * math.pi / orient), math.sin(k * math.pi / orient)
            if order == 0:
                want = fma32(f32(sn), b1, f32(cs) * b0)
            else:
                want = fma32(f32(cs * cs), b0, f32(sn * sn) * b1)
            got = d[order * orient + k]
            assert np.array_equal(got[sure], want[sure]), (order, k, int((got != want)[sure].sum()))
