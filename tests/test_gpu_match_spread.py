"""The pair call's two forms of the match transforms: a workgroup per interest
point and channel (few points, taken where the workspace has its scratch) and a
workgroup per point.  Same products, summed in the same order."""
import ctypes

import numpy as np
import pytest

from paper_2202_13347_amd import sfoc as S
from paper_2202_13347_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def run(reg, ws_bytes, ref, sen, ips, prior):
    Hr, Wr, Hs, Ws, n, m, r = reg.shape
    reg.ws.fill_(0x7f)
    reg.ncc.fill_(7.0)
    rc = S.lib().sfoc_register_cps(S._ptr(ref), Hr, Wr, ref.stride(0), S._ptr(sen), Hs, Ws, sen.stride(0), S._ptr(ips),
                                   S._ptr(prior), n, m, r, ctypes.byref(reg.p), S._ptr(reg.ncc), S._ptr(reg.cps),
                                   S._ptr(reg.ws), ws_bytes, S._stream(None))
    torch.cuda.synchronize()
    return rc, reg.ncc.cpu().numpy(), S.cps_to_numpy(reg.cps)


# m, r: each transform side; n: one, ragged, the most that the form takes
@pytest.mark.parametrize("m,r,n,dtype,prior,orient", [
    (32, 10, 1, S.DTYPE_F32, False, 8), (41, 11, 33, S.DTYPE_F32, True, 6), (24, 18, 9, S.DTYPE_BF16, True, 2),
    (49, 17, 17, S.DTYPE_F16, True, 6), (64, 32, 128, S.DTYPE_F32, False, 8),
    (65, 47, 5, S.DTYPE_BF16, False, 3), (96, 48, 7, S.DTYPE_F32, True, 8),
])
def test_forms_agree(m, r, n, dtype, prior, orient):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print("spread", m, r, n, dtype, prior, orient, flush=True)
    H, W = 2 * (m + 2 * r) + 33, 2 * (m + 2 * r) + 50
    pr = synth.make_pair(31 + m, (H, W), 3.0)
    rng = np.random.default_rng(n)
    lo = (m + 1) // 2 + r + 4
    ips = np.stack([rng.integers(lo, H - lo, n), rng.integers(lo, W - lo, n)], 1).astype(np.int32)
    if n > 1:
        ips[n // 2] = 2   # out of bounds
    d_prior = torch.from_numpy(rng.integers(-3, 4, (n, 2)).astype(np.int32)).cuda() if prior else None
    ref, sen, d_ips = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (pr.ref, pr.sen, ips))
    p = S.params(n_orient=orient, dtype=dtype)
    reg = S.Registrar(H, W, H, W, n, m, r, p, want_ncc=True)
    L = next(s for s in (64, 128, 160, 192) if m + 2 * r <= s)
    scratch = n * 2 * orient * (4 * L * L + 48)
    least = reg.wsb - scratch
    rc, ncc, cps = run(reg, reg.wsb, ref, sen, d_ips, d_prior)
    assert rc == S.SFOC_OK
    rc, want, wcps = run(reg, least, ref, sen, d_ips, d_prior)
    assert rc == S.SFOC_OK
    assert run(reg, least - 1, ref, sen, d_ips, d_prior)[0] == S.SFOC_E_WORKSPACE
    # the spectra's sums are the same; the template sums (float64) may differ in
    # their last bit, so a score by one float32 rounding
    np.testing.assert_allclose(ncc, want, rtol=0, atol=2.0 ** -23)
    for f in ("sen_row", "sen_col", "dy", "dx", "flags"):
        np.testing.assert_array_equal(cps[f], wcps[f])


def test_scratch_bounds():
    """No scratch for more points than the form is taken for, or few channels."""
    p = S.params(n_orient=8)
    size = lambda n, q=p: S.register_workspace(600, 600, 600, 600, n, 64, 32, q)
    assert size(128) - size(129) > 128 * 16 * 4 * 128 * 128 - (1 << 20)
    assert size(16, S.params(n_orient=1)) < size(16, S.params(n_orient=2)) - 16 * 4 * 4 * 128 * 128
