"""The head's activations bit for bit: every pre-activation is one chain of
float32 fused multiply-adds from the bias, a convolution's over input channels
and then taps, a fully connected layer's over its inputs.  The ReLUs' decisions,
and with them what a whole unit adds to a gradient, follow from those bits: with
biases that put a unit of every channel within rounding of zero, gradients in
float64 over the emulated activations' masks have to agree."""
import numpy as np
import pytest

from oracle import head_oracle as H
from paper_2202_13347_amd import sfoc as S
from paper_2202_13347_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def fma32(a, b, c):
    """float32 fused multiply-add: the product is exact in float64, the sum is
    rounded to odd there (by its exact error) before its rounding to float32."""
    p, c = a.double() * b.double(), c.double()
    s = p + c
    t = s - p
    err = (p - (s - t)) + (c - t)
    even = (s.view(torch.int64) & 1) == 0
    s = torch.where((err != 0) & even, torch.nextafter(s, torch.copysign(torch.full_like(s, np.inf), err)), s)
    return s.float()


def conv_chain(x, w, b, stride):
    """Pre-activations: w (O, C, 3, 3), b (O) or None (products alone, float64)."""
    n, C, side, _ = x.shape
    so = (side - 1) // stride + 1
    xp = torch.nn.functional.pad(x, (1, 1, 1, 1))
    acc = torch.zeros((n, w.shape[0], so, so), dtype=torch.float64 if b is None else torch.float32, device=x.device)
    acc = acc if b is None else acc + b[None, :, None, None]
    for c in range(C):
        for i in range(3):
            for j in range(3):
                v = xp[:, c, i:i + stride * (so - 1) + 1:stride, j:j + stride * (so - 1) + 1:stride][:, None]
                k = w[:, c, i, j][None, :, None, None]
                acc = acc + k.double() * v.double() if b is None else fma32(k, v, acc)
    return acc


def fc_chain(x, w, b):
    acc = torch.zeros((x.shape[0], w.shape[0]), dtype=torch.float64 if b is None else torch.float32, device=x.device)
    acc = acc if b is None else acc + b[None]
    for k in range(x.shape[1]):
        u, v = w[None, :, k], x[:, None, k]
        acc = acc + u.double() * v.double() if b is None else fma32(u, v, acc)
    return acc


def near_zero(z):
    """Biases that put one entry of every channel within rounding of zero: of
    z (bias-free pre-activations; channels second) the median one."""
    return -z.transpose(0, 1).flatten(1).median(1).values.float()


def emulate(theta, crops, stats, place=False):
    """(outputs, activations, parameters): with `place` the biases of conv2,
    conv3, conv4 and fc1 are chosen layer by layer by near_zero."""
    P = {k: dev(v.astype(np.float32)) for k, v in H.unpack(theta).items()}
    q = {k: dev(H.bf16(v).astype(np.float32)) for k, v in H.unpack(theta).items() if k.endswith("w")}
    acts = [dev(crops)[:, None]]
    for k, (_, _, stride) in enumerate(H.CONVS):
        w, b = q[f"conv{k + 1}.w"], f"conv{k + 1}.b"
        if place and k:
            P[b] = near_zero(conv_chain(acts[-1], w, None, stride))
        acts.append(conv_chain(acts[-1], w, P[b], stride).clamp_min(0))
    x = torch.cat([acts[-1].flatten(1), dev(stats)], 1)
    if place:
        P["fc1.b"] = near_zero(fc_chain(x, q["fc1.w"], None))
    h = fc_chain(x, q["fc1.w"], P["fc1.b"]).clamp_min(0)
    out = fc_chain(h, q["fc2.w"], P["fc2.b"])
    return (out.cpu().numpy(), [a.cpu().numpy() for a in acts + [x, h]],
            H.pack({k: v.cpu().numpy() for k, v in P.items()}).astype(np.float32))


def gradients(theta, out, acts, label, target):
    """float64 gradients with the masks of the emulated activations."""
    q = {k: H.bf16(v) if k.endswith("w") else v for k, v in H.unpack(theta).items()}
    do = H.loss_grad(out.astype(np.float64), label, target[:, 0], target[:, 1])
    x, h = acts[5].astype(np.float64), acts[6].astype(np.float64)
    g = {"fc2.w": do.T @ h, "fc2.b": do.sum(0)}
    dh = do @ q["fc2.w"] * (h > 0)
    g["fc1.w"], g["fc1.b"] = dh.T @ x, dh.sum(0)
    da = (dh @ q["fc1.w"])[:, :800].reshape(acts[4].shape)
    for k in (3, 2, 1, 0):
        dz = da * (acts[k + 1] > 0)
        da, g[f"conv{k + 1}.w"], g[f"conv{k + 1}.b"] = H.conv_backward(
            acts[k].astype(np.float64), q[f"conv{k + 1}.w"], dz, H.CONVS[k][2])
    return g


def batch(n, seed):
    rng = np.random.default_rng(seed)
    th = synth.head_init_params(7) + rng.normal(0, 0.02, S.HEAD_PARAMS).astype(np.float32)
    crops = rng.uniform(-1, 1, (n, 33, 33)).astype(np.float32)
    stats = rng.uniform(-1, 1, (n, 8)).astype(np.float32)
    label = (rng.random(n) < 0.6).astype(np.float32)
    label[0] = 1.0
    target = rng.uniform(-0.6, 0.6, (n, 2)).astype(np.float32)
    return th, crops, stats, label, target


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# One sample, a few with units within rounding of zero, a workgroup per sample
# (in the batch of 256 a unit of conv2 lies at 1.4e-8) and one with two samples.
# The gradient sums are float32 chains of at most 33 * 33 products and then the
# batch: errors of sqrt(1089) 2^-24 = 2e-6 of the block's norm, ten times that
# where terms cancel.  (A unit on the other side of zero: 5e-4 and more.)
@pytest.mark.parametrize("n, place", [(1, False), (5, True), (256, False), (257, False)])
def test_chains(n, place):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print(f"head order n={n} place={place}", flush=True)
    th, crops, stats, label, target = batch(n, 100 + n)
    out, acts, th = emulate(th, crops, stats, place)
    got = S.Head(th).forward(dev(crops), dev(stats)).cpu().numpy()
    np.testing.assert_array_equal(got, out)
    want = gradients(th, out, acts, label, target)
    _, grad = S.Head(th).train_step(dev(crops), dev(stats), dev(label), dev(target), lr=0.0, want_grad=True)
    got = H.unpack(grad.cpu().numpy())
    for name, _ in H.layout():
        err = np.linalg.norm(got[name] - want[name]) / np.linalg.norm(want[name])
        assert err <= 2e-5, (name, err)
