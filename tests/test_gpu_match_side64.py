"""Side-64 transforms: the surfaces' bits.  At side 64 two products of the 8-point
codelet round differently in the upper half of a pass's row pairs or columns.  The
digests are of the surfaces that the kernels gave when the compiler chose the roundings;
descriptor values are whole 256ths, so the integral images are exact in any order."""
import hashlib

import numpy as np
import pytest

from paper_2202_13347_amd import sfoc as S

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

H, W, N = 150, 190, 40


def points(m, r, H, W):
    rng = np.random.default_rng(m)
    lo = m // 2 + r + 1
    ips = np.stack([rng.integers(lo, H - lo, N), rng.integers(lo, W - lo, N)], 1)
    return torch.from_numpy(ips.astype(np.int32)).cuda()


def digest(ncc):
    a = ncc.cpu().numpy()
    assert np.isfinite(a).all()
    return hashlib.sha256(a.tobytes()).hexdigest()[:16]


# Windows of 31 to 64 samples: up to half, three quarters and all of the side.
CALLS = {
    ("float32", 8, 17): "6ec11620b521af86", ("float32", 32, 16): "70b7e99664b5c3a3",
    ("float32", 13, 25): "131aa467435e2733", ("float32", 5, 13): "6709b4e7256211ed",
    ("bfloat16", 8, 17): "88f277e7628a7c6a", ("bfloat16", 32, 16): "088d752b0271bca8",
    ("bfloat16", 13, 25): "115d6ec11a34b482", ("bfloat16", 16, 16): "1ac6cbdbc281f09f",
    ("float16", 8, 17): "6ec11620b521af86", ("float16", 32, 16): "70b7e99664b5c3a3",
    ("float16", 13, 25): "131aa467435e2733", ("float16", 16, 16): "a3c6146446cf84ab",
}


@pytest.mark.parametrize("dtype,m,r", list(CALLS))
def test_call(dtype, m, r):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print("side 64", dtype, m, r, flush=True)
    rng = np.random.default_rng(7)
    ref, sen = (rng.integers(-255, 256, (6, H, W)) / 256.0 for _ in range(2))
    integ = []
    for a in (ref.sum(0), (ref * ref).sum(0)):
        t = np.zeros((H + 1, W + 1))
        t[1:, 1:] = a.cumsum(0).cumsum(1)
        integ.append(torch.from_numpy(t).cuda())
    ds, dr = (torch.from_numpy(a).cuda().to(getattr(torch, dtype)).contiguous() for a in (sen, ref))
    ncc = S.fastncc_match(ds, dr, *integ, points(m, r, H, W), m, r, want_ncc=True)[1]
    assert digest(ncc) == CALLS[dtype, m, r]


# A plan's FFT form with templates past half of the side (a call takes the direct form
# for these types there).
PLANS = {
    (S.DTYPE_BF16, 48, 8): "9eca344b2e21c65e",
    (S.DTYPE_BF16, 40, 5): "94ef056da892620c",
    (S.DTYPE_F16, 48, 8): "d091f03706001775",
}


@pytest.mark.parametrize("dtype,m,r", list(PLANS))
def test_plan(dtype, m, r):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print("side 64 plan", dtype, m, r, flush=True)
    rng = np.random.default_rng(8)
    ref, sen = (torch.from_numpy((rng.integers(0, 256, (H, W)) / 256.0).astype(np.float32)).cuda() for _ in range(2))
    plan = S.Plan([dict(ref=ref, sen=sen, ips=points(m, r, H, W), m=m, r=r, fft_side=64)],
                  S.params(n_orient=4, dtype=dtype), want_ncc=True)
    plan()
    got = digest(plan.ncc[0])
    plan.close()
    assert got == PLANS[dtype, m, r]
