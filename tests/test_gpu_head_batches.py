"""The head's network at the batch sizes where its work is split differently:
one sample, a workgroup per sample up to the largest grid (256) and a workgroup
that takes a second sample (257).  Loss, gradients and outputs against the FP64 oracle, and the training step against
itself bit for bit."""
import numpy as np
import pytest

from oracle import head_oracle as H
from paper_2202_13347_amd import sfoc as S
from paper_2202_13347_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# FP32 sums of at most 2^17 rounded products in chains of at most 2^10: relative
# errors below 2^10 eps / 2 = 3e-5 for a sum without cancellation; the blocks'
# norms are held to the 1e-4 of the other gradient tests, the outputs to theirs.
@pytest.mark.parametrize("n", [1, 256, 257])
def test_batch_sizes(n):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print(f"head batch n={n}", flush=True)
    rng = np.random.default_rng(100 + n)
    th = synth.head_init_params(7) + rng.normal(0, 0.02, S.HEAD_PARAMS).astype(np.float32)
    crops = rng.uniform(-1, 1, (n, 33, 33)).astype(np.float32)
    stats = rng.uniform(-1, 1, (n, 8)).astype(np.float32)
    label = (rng.random(n) < 0.6).astype(np.float32)
    label[0] = 1.0
    target = rng.uniform(-0.6, 0.6, (n, 2)).astype(np.float32)
    th64 = th.astype(np.float64)

    out = S.Head(th).forward(dev(crops), dev(stats)).cpu().numpy()
    want, _ = H.forward(th64, crops, stats, quantise=True)
    np.testing.assert_allclose(out, want, rtol=1e-4, atol=1e-4 * np.abs(want).max())

    loss, grad = S.Head(th).train_step(dev(crops), dev(stats), dev(label), dev(target), lr=0.0, want_grad=True)
    L, wg = H.backward(th64, crops, stats, label, target[:, 0], target[:, 1], quantise=True)
    assert float(loss) == pytest.approx(L, rel=1e-5)
    g = grad.cpu().numpy()
    o = 0
    for name, shape in H.layout():
        k = int(np.prod(shape))
        err = np.linalg.norm(g[o:o + k] - wg[o:o + k]) / max(np.linalg.norm(wg[o:o + k]), 1e-12)
        assert err <= 1e-4, (name, err)
        o += k
    loss2, grad2 = S.Head(th).train_step(dev(crops), dev(stats), dev(label), dev(target), lr=0.0, want_grad=True)
    assert float(loss2) == float(loss)
    np.testing.assert_array_equal(grad2.cpu().numpy(), g)
