"""How the describe kernels store a run of pixels: as one vector, pixel by pixel, and past
the row's end.  Descriptors have the same bits wherever they are written to, nothing
beside them is written, and the integral images are those of the stored values."""
import numpy as np
import pytest

from paper_2202_13347_amd import sfoc as S

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# Widths of whole runs (the last tile ends inside a run's vector, or has runs past the
# image), and of one, two and three pixels more.
@pytest.mark.parametrize("H,W", [(32, 64), (33, 31), (40, 36), (13, 41), (65, 98), (100, 132)])
@pytest.mark.parametrize("dtype", [S.DTYPE_F32, S.DTYPE_BF16, S.DTYPE_F16])
@pytest.mark.parametrize("bank", [dict(n_orient=8), dict(n_orient=3), dict(n_orient=4, second_order=False)])
def test_forms(H, W, dtype, bank):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print("describe forms", H, W, dtype, bank, flush=True)
    rng = np.random.default_rng(H * W)
    img = torch.from_numpy(rng.random((H, W)).astype(np.float32)).cuda()
    p = S.params(dtype=dtype, **bank)
    z = S.check_params(p)
    n = z * H * W
    want = None
    for off in range(3):   # elements past a vector's alignment
        buf = torch.full((n + 8,), 7.0, dtype=S._desc_torch_dtype(dtype), device="cuda")
        desc = buf[off:off + n].view(z, H, W)
        _, i1, i2 = S.describe(img, p, out=desc)
        assert (buf[:off] == 7).all() and (buf[off + n:] == 7).all()
        if want is None:
            want = desc.clone()
            d = want.double().cpu().numpy()
            assert np.isfinite(d).all()
            for got, v in ((i1, d), (i2, d * d)):
                ref = np.zeros((H + 1, W + 1))
                ref[1:, 1:] = v.sum(0).cumsum(0).cumsum(1)
                # both sides add fewer than z + H + W times in sequence, in float64
                bound = 2 * (z + H + W) * 2.0 ** -53 * np.abs(v).sum()
                assert np.abs(got.cpu().numpy() - ref).max() <= bound
            first = (i1, i2)
        assert torch.equal(desc, want)
        assert torch.equal(i1, first[0]) and torch.equal(i2, first[1])
