"""Outlier rejection at the candidate counts where the final kernel's batches
end: fewer candidates than threads, whole and ragged batches of 512 and 2048."""
import pytest

from oracle import ransac_oracle as R
from tests.test_gpu_ransac import compare, records

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# candidates: no record is flagged out, so n of them
@pytest.mark.parametrize("model", [R.AFFINE, R.PROJECTIVE])
@pytest.mark.parametrize("n", [5, 63, 511, 512, 513, 2047, 2049])
def test_batch_edges(n, model):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print("ransac", n, model, flush=True)
    c, _ = records(700 + n, n, 1500, model, frac_bad=0.25 if n > 8 else 0.0, frac_flagged=0.0)
    compare(c, None, model, 64, 2, (1500, 1500, 1500, 1500))
