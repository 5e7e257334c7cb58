"""The pair call's spread form against its fused form where the last bit of the
template sums R_T and R_TT shows: descriptors whose variance is far below their
mean square, so that R_TT - R_T^2 / (m m z) cancels.  Both forms add in one order,
so surfaces and records are the same bits; which form ran is seen from the
workspace."""
import ctypes

import numpy as np
import pytest

from paper_2202_13347_amd import sfoc as S

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def flat_pair(size, seed, noise):
    """exp(k (x + y)): Gx = Gy and Gxx = Gyy, so with two orientations all four
    channels are 1 / sqrt 2 but for the noise."""
    rng = np.random.default_rng(seed)
    y, x = np.mgrid[:size, :size].astype(np.float64)
    k = 2.0 / size
    out = []
    for _ in range(2):
        out.append((np.exp(k * (x + y)) * (1 + noise * rng.standard_normal((size, size)))).astype(np.float32))
    return out


def item_bytes(side, z):
    return z * (4 * side * side + 48)


# Each side; at 160 templates of one and two rounds of row pairs; the most points
# that the form is taken for, by number and (192, z = 16) by size.
@pytest.mark.parametrize("m,r,n,dtype,orient", [
    (32, 10, 17, S.DTYPE_F32, 2), (33, 15, 512, S.DTYPE_F32, 2), (64, 32, 33, S.DTYPE_F32, 2),
    (63, 20, 128, S.DTYPE_F32, 8), (65, 47, 96, S.DTYPE_F32, 2), (141, 9, 9, S.DTYPE_F32, 3),
    (96, 48, 5, S.DTYPE_F32, 2), (64, 50, 9, S.DTYPE_BF16, 6), (48, 8, 17, S.DTYPE_F32, 4),
    (64, 64, 67, S.DTYPE_F32, 8), (65, 17, 9, S.DTYPE_F16, 2),
])
def test_same_bits(m, r, n, dtype, orient):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print("spread sums", m, r, n, dtype, orient, flush=True)
    M = m + 2 * r
    side, size = next(s for s in (64, 128, 160, 192) if M <= s), 2 * M + 40
    p = S.params(n_orient=orient, dtype=dtype)
    rng = np.random.default_rng(n)
    ref, sen = (torch.from_numpy(a).cuda() for a in flat_pair(size, m, 3e-6 if dtype == S.DTYPE_F32 else 3e-3))
    ips = torch.from_numpy(rng.integers(M // 2 + 1, size - M // 2 - 1, (n, 2)).astype(np.int32)).cuda()
    reg = S.Registrar(size, size, size, size, n, m, r, p, want_ncc=True)
    least = reg.wsb - n * item_bytes(side, 2 * orient)

    def run(ws_bytes):
        reg.ws.fill_(0x7f)
        reg.ncc.fill_(7.0)
        rc = S.lib().sfoc_register_cps(S._ptr(ref), size, size, size, S._ptr(sen), size, size, size, S._ptr(ips), None,
                                       n, m, r, ctypes.byref(reg.p), S._ptr(reg.ncc), S._ptr(reg.cps), S._ptr(reg.ws),
                                       ws_bytes, S._stream(None))
        torch.cuda.synchronize()
        assert rc == S.SFOC_OK
        return reg.ncc.cpu().numpy(), S.cps_to_numpy(reg.cps), bool((reg.ws[least:] != 0x7f).any())

    ncc, cps, used = run(reg.wsb)
    want, wcps, unused = run(least)
    assert used and not unused
    assert len(np.unique(want)) > n
    np.testing.assert_array_equal(ncc, want)
    for f in wcps.dtype.names:
        np.testing.assert_array_equal(cps[f], wcps[f], err_msg=f)


@pytest.mark.parametrize("m,r,orient,most", [(32, 10, 8, 512), (64, 32, 8, 128), (64, 48, 4, 96), (64, 64, 4, 96),
                                             (64, 64, 8, 67)])
def test_most_points(m, r, orient, most):
    """Scratch for `most` points and not for one more."""
    p = S.params(n_orient=orient)
    side = next(s for s in (64, 128, 160, 192) if m + 2 * r <= s)
    size = lambda n: S.register_workspace(600, 600, 600, 600, n, m, r, p)
    assert size(most) - size(most + 1) > most * item_bytes(side, 2 * orient) - (1 << 20)
