"""The work this library is used for, as cases that can be timed.

One kind per public entry point: the pair call (`Registrar`, what most
programs run), dense descriptors (`describe`), template matching on
descriptors a program already holds (`fastncc_match`), the batched plan
(`Plan`), the learned head's training step and its inference, outlier
rejection (`Ransac`), resampling (`rectify`) and interest-point detection
(`Detector`).  Sizes are those of the workload recipes in
`paper_2202_13347_amd.synth` and of `bench.py`; `draw` spreads them over
what lies between, odd sizes among them.

Inputs are drawn on the GPU from the seed: piecewise-constant scenes seen
through two different intensity responses, blurred, shifted, with additive
noise and speckle on the sensed image, as `synth.make_pair` describes them.
"""
from __future__ import annotations

import math
import os

import numpy as np
import torch

from paper_2202_13347_amd import sfoc as S

DEV = "cuda"
DTYPES = {"f32": (S.DTYPE_F32, torch.float32), "bf16": (S.DTYPE_BF16, torch.bfloat16),
          "f16": (S.DTYPE_F16, torch.float16)}
ES = {"f32": 4, "bf16": 2, "f16": 2}
# orientations, first- and second-order standard deviations of the two presets
BANK = {"baseline": (8, (1.0, 2.0, 3.0), (1.0, 2.0, 3.0)), "paper": (6, (0.6, 0.8, 1.0), (1.5,))}
SD1, SD2, EPS, RATES = 1.0, 1.5, 1e-8, (1, 2, 3)
Q = 3   # reach of the dilated smoothing


def listed():
    return [
        # The smallest registration: a 256 x 256 pair with a 4 x 4 grid (the
        # `small` recipe), surfaces kept.  Latency and launches count.
        dict(name="pair_small", kind="pair", Hr=256, Wr=256, Hs=256, Ws=256, n=16, m=32, r=10, dtype="f32",
             preset="baseline", prior=False, ncc=True, looks=0),
        # An ordinary pair of uneven, odd-sided images with an odd template, a
        # prior per interest point, the paper's filter bank and float16 storage.
        dict(name="pair_ragged", kind="pair", Hr=613, Wr=771, Hs=597, Ws=805, n=119, m=49, r=17, dtype="f16",
             preset="paper", prior=True, ncc=True, looks=4),
        # The benchmark scene: 2048 x 2048, 400 interest points.
        dict(name="pair_scene", kind="pair", Hr=2048, Wr=2048, Hs=2048, Ws=2048, n=400, m=64, r=32, dtype="f32",
             preset="baseline", prior=False, ncc=False, looks=4),
        # The largest: a full satellite scene, 5000 interest points, bfloat16
        # descriptors (the `large` recipe).
        dict(name="pair_large", kind="pair", Hr=10000, Wr=10000, Hs=10000, Ws=10000, n=5000, m=64, r=48,
             dtype="bf16", preset="baseline", prior=False, ncc=False, looks=4),
        # Dense descriptors of a whole image with their integral images, for a
        # program that matches against them later.
        dict(name="describe_scene", kind="describe", H=2048, W=2048, dtype="f32", preset="baseline"),
        # Small search windows on 16-bit descriptors (a good prior), integral
        # images per window.
        dict(name="match_small_windows", kind="match", H=2048, W=2048, n=400, m=32, r=10, dtype="bf16", window=True),
        # Serving: several uneven pairs as one graph-replayed plan (the `batch`
        # recipe's template sides and radii).
        dict(name="plan_batch", kind="plan", pairs=12, side_lo=512, side_hi=2048, n_lo=50, n_hi=250, dtype="f32",
             spec=7),
        # One optimiser step of the learned head at its training batch size.
        dict(name="head_train", kind="head_train", n=256),
        # The learned head on the control points of a scene: features from the
        # surfaces, network, decision.
        dict(name="head_infer", kind="head_infer", H=2048, W=2048, n=400, m=64, r=32, dtype="f32"),
        # Outlier rejection over the control points of a large scene.
        dict(name="ransac_large", kind="ransac", n=5041, n_hyp=4096, model="projective", n_refine=2, size=10000),
        # Resampling of a full scene into the reference grid.
        dict(name="rectify_large", kind="rectify", Hs=10000, Ws=10000, Ho=10000, Wo=10000, pad=0),
        # Interest points of a full scene, one per block.
        dict(name="fast_large", kind="fast", H=10000, W=10000, nby=71, nbx=71, per=1, margin=80, threshold=0.05),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: a kind, then sizes over its range (logarithmically)."""
    kind = rng.choice(["pair", "pair", "pair", "describe", "match", "plan", "head_train", "head_infer", "ransac",
                       "rectify", "fast"])
    if kind == "pair":
        m = rng.choice([32, 48, 64, rng.randrange(24, 97), 96])
        r = rng.choice([10, 16, 32, 48, rng.randrange(8, 65)])
        lo = 2 * (m + r) + 40
        Hs, Ws = _log_int(rng, max(256, lo), 4096), _log_int(rng, max(256, lo), 4096)
        Hr, Wr = (Hs, Ws) if rng.random() < 0.5 else (Hs + rng.randrange(0, 40), Ws + rng.randrange(0, 40))
        return dict(kind="pair", Hr=Hr, Wr=Wr, Hs=Hs, Ws=Ws, n=_log_int(rng, 16, 1000), m=m, r=r,
                    dtype=rng.choice(["f32", "f32", "bf16", "f16"]), preset=rng.choice(["baseline", "baseline", "paper"]),
                    prior=rng.random() < 0.3, ncc=rng.random() < 0.5, looks=rng.choice([0, 4]))
    if kind == "describe":
        return dict(kind="describe", H=_log_int(rng, 200, 5000), W=_log_int(rng, 200, 5000),
                    dtype=rng.choice(["f32", "bf16", "f16"]), preset=rng.choice(["baseline", "paper"]))
    if kind == "match":
        m, r = rng.choice([(24, 6), (32, 10), (48, 12), (64, 15), (64, 32), (96, 32)])
        return dict(kind="match", H=_log_int(rng, 400, 2500), W=_log_int(rng, 400, 2500), n=_log_int(rng, 16, 1600),
                    m=m, r=r, dtype=rng.choice(["bf16", "f16", "f32"]), window=rng.random() < 0.5)
    if kind == "plan":
        return dict(kind="plan", pairs=rng.randrange(3, 17), side_lo=512, side_hi=_log_int(rng, 700, 2600), n_lo=50,
                    n_hi=_log_int(rng, 80, 400), dtype=rng.choice(["f32", "f32", "bf16"]), spec=rng.randrange(1 << 30))
    if kind == "head_train":
        return dict(kind="head_train", n=_log_int(rng, 32, 1024))
    if kind == "head_infer":
        m, r = rng.choice([(32, 10), (48, 16), (64, 32)])
        return dict(kind="head_infer", H=_log_int(rng, 400, 2500), W=_log_int(rng, 400, 2500),
                    n=_log_int(rng, 16, 1600), m=m, r=r, dtype=rng.choice(["f32", "bf16"]))
    if kind == "ransac":
        return dict(kind="ransac", n=_log_int(rng, 50, 16000), n_hyp=_log_int(rng, 256, 8192),
                    model=rng.choice(["affine", "projective"]), n_refine=rng.choice([0, 1, 2, 4]),
                    size=rng.choice([2048, 10000]))
    if kind == "rectify":
        return dict(kind="rectify", Hs=_log_int(rng, 300, 10000), Ws=_log_int(rng, 300, 10000),
                    Ho=_log_int(rng, 300, 10000), Wo=_log_int(rng, 300, 10000), pad=rng.choice([0, 0, 5]))
    nb = _log_int(rng, 4, 71)
    return dict(kind="fast", H=_log_int(rng, 512, 10000), W=_log_int(rng, 512, 10000), nby=nb, nbx=nb + rng.randrange(5),
                per=rng.choice([1, 1, 2, 5]), margin=rng.choice([3, 40, 64]), threshold=rng.choice([0.05, 0.1]))


# ---- inputs ----------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) & 0x7fffffff)


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV)


def _field(g, H, W, cell):
    """Smooth random field in [0, 1]: a coarse uniform grid, bilinear."""
    c = _rand(g, 1, 1, H // cell + 3, W // cell + 3)
    return torch.nn.functional.interpolate(c, size=(H, W), mode="bilinear", align_corners=True)[0, 0]


def _blur(x):
    """Gaussian of standard deviation 1 (radius 3), edges clamped."""
    t = [math.exp(-0.5 * k * k) for k in range(-3, 4)]
    s = sum(t)
    for axis in (0, 1):
        n = x.shape[axis]
        idx = torch.arange(-3, n + 3, device=DEV).clamp_(0, n - 1)
        e = x.index_select(axis, idx)
        x = sum((t[k] / s) * e.narrow(axis, k, n) for k in range(7))
    return x


def _images(g, Hr, Wr, Hs, Ws, max_shift, looks):
    """(reference, sensed) float32 images and the shift (dy, dx)."""
    pad = int(max_shift) + 4
    H, W = max(Hr, Hs) + 2 * pad, max(Wr, Ws) + 2 * pad
    a = (_field(g, H, W, 31) * 23.0).to(torch.int64)
    b = (_field(g, H, W, 13) * 3.0).to(torch.int64)
    lab = a * 3 + b                                  # regions: level sets of two fields
    k = 24 * 3
    val = _rand(g, k)
    scene = val[lab] + 0.2 * (_field(g, H, W, 16) - 0.5)
    # per region a cubic response, scaled to its range on [0, 1], half reversed
    c = _rand(g, k, 4) * 4.0 - 2.0
    v = torch.linspace(0, 1, 65, device=DEV)
    y = c[:, :1] + v * (c[:, 1:2] + v * (c[:, 2:3] + v * c[:, 3:4]))
    lo, span = y.min(1).values, (y.max(1).values - y.min(1).values).clamp_min(0.05)
    flip = _rand(g, k) < 0.5
    q = c[lab]
    s = (q[..., 0] + scene * (q[..., 1] + scene * (q[..., 2] + scene * q[..., 3])) - lo[lab]) / span[lab]
    s = torch.where(flip[lab], 1.0 - s, s)
    del q, lab
    scene, s = _blur(scene), _blur(s)
    d = ((_rand(g, 2) * 2.0 - 1.0) * max_shift).tolist()
    iy, ix = math.floor(d[0]), math.floor(d[1])
    fy, fx = d[0] - iy, d[1] - ix
    t = s[pad + iy:pad + iy + Hs + 1, pad + ix:pad + ix + Ws + 1]
    t = (1 - fy) * t[:-1] + fy * t[1:]
    sen = (1 - fx) * t[:, :-1] + fx * t[:, 1:]
    sen = sen + 0.05 * torch.randn(Hs, Ws, generator=g, device=DEV)
    if looks:                                        # mean of `looks` unit exponentials
        e = sum(-torch.log1p(-_rand(g, Hs, Ws)) for _ in range(looks)) / looks
        sen = sen * e
    return scene[pad:pad + Hr, pad:pad + Wr].contiguous(), sen.contiguous(), d


def _points(g, n, Hs, Ws, Hr, Wr, m, r, slack=0):
    """n uniform interest points whose template and search window fit."""
    b = (m + 1) // 2 + r + slack
    H, W = min(Hs, Hr), min(Ws, Wr)
    y = b + (_rand(g, n).double() * max(1, H - 2 * b)).to(torch.int32)
    x = b + (_rand(g, n).double() * max(1, W - 2 * b)).to(torch.int32)
    return torch.stack([y, x], 1).to(torch.int32).contiguous()


def _pair_inputs(c, seed):
    g = _gen(seed)
    slack = 3 if c["prior"] else 0
    ref, sen, d = _images(g, c["Hr"], c["Wr"], c["Hs"], c["Ws"], max(1.0, 0.8 * c["r"]), c["looks"])
    ips = _points(g, c["n"], c["Hs"], c["Ws"], c["Hr"], c["Wr"], c["m"], c["r"], slack)
    prior = None
    if c["prior"]:
        prior = (torch.floor(_rand(g, c["n"], 2) * (2 * slack + 1)) - slack).to(torch.int32).contiguous()
    return ref, sen, ips, prior


def _plan_specs(c):
    """Sizes of the plan's pairs (fixed by the case, not by the seed)."""
    rs = np.random.RandomState(c["spec"] & 0x7fffffff)
    out = []
    for k in range(c["pairs"]):
        side = int(round(math.exp(rs.uniform(math.log(c["side_lo"]), math.log(c["side_hi"])))))
        m, r = int(rs.choice([48, 64, 96])), int(rs.choice([16, 32, 64]))
        n = int(rs.randint(c["n_lo"], c["n_hi"] + 1))
        out.append(dict(Hr=side, Wr=side, Hs=side, Ws=side, n=n, m=m, r=r, prior=False, looks=4 if k % 2 else 0,
                        dtype=c["dtype"], preset="baseline"))
    return out


def _plan_inputs(c, seed):
    return [(s, *_pair_inputs(s, seed * 131 + k)) for k, s in enumerate(_plan_specs(c))]


def _match_inputs(c, seed):
    """Descriptors of a pair (plain torch), integral images of the reference
    and interest points."""
    g = _gen(seed)
    ref, sen, _ = _images(g, c["H"], c["W"], c["H"], c["W"], max(1.0, 0.8 * c["r"]), 4)
    ips = _points(g, c["n"], c["H"], c["W"], c["H"], c["W"], c["m"], c["r"])
    dt = DTYPES[c["dtype"]][1]
    dref = _sfoc64(ref, "baseline").float().to(dt).contiguous()
    dsen = _sfoc64(sen, "baseline").float().to(dt).contiguous()
    return dref, dsen, ips


def _integrals(desc):
    H, W = desc.shape[1:]
    out = []
    for p in (1, 2):
        i = torch.zeros(H + 1, W + 1, dtype=torch.float64, device=DEV)
        s = torch.zeros(H, W, dtype=torch.float64, device=DEV)
        for ch in desc:
            s += ch.double() ** p
        i[1:, 1:] = s.cumsum(0).cumsum(1)
        out.append(i)
    return out


HEAD_SHAPES = [(32, 1, 3, 3), (32,), (32, 32, 3, 3), (32,), (32, 32, 3, 3), (32,), (32, 32, 3, 3), (32,), (32, 808),
               (32,), (3, 32), (3,)]


def _head_params():
    """The trained parameters that ship with the package."""
    path = os.path.join(os.path.dirname(os.path.abspath(S.__file__)), "head_params.f32")
    return torch.from_numpy(np.fromfile(path, dtype="<f4").copy())


def _head_batch(c, seed):
    """Surface crops with one peak over correlated noise, their statistics,
    labels and offsets; Adam moments of a run that is under way."""
    g = _gen(seed)
    n = c["n"]
    ax = torch.arange(-16, 17, device=DEV, dtype=torch.float32)
    off = _rand(g, n, 2) - 0.5
    w = 1.5 + 2.5 * _rand(g, n, 1, 1)
    amp = 0.2 + 0.6 * _rand(g, n, 1, 1)
    bump = torch.exp(-((ax[None, :, None] - off[:, :1, None]) ** 2 + (ax[None, None, :] - off[:, 1:, None]) ** 2)
                     / (2 * w * w))
    noise = torch.nn.functional.interpolate(_rand(g, n, 1, 12, 12) - 0.5, size=(33, 33), mode="bilinear",
                                            align_corners=True)[:, 0]
    crops = (amp * bump + 0.3 * noise).contiguous()
    stats = torch.stack([crops[:, 16, 16], crops.flatten(1).amax(1) * 0.9, crops.flatten(1).mean(1),
                         crops.flatten(1).std(1), 0.05 + 0.1 * _rand(g, n), 0.05 + 0.1 * _rand(g, n),
                         0.2 + 0.1 * _rand(g, n), -0.05 * _rand(g, n)], 1).contiguous()
    label = (_rand(g, n) < 0.7).float()
    target = ((_rand(g, n, 2) - 0.5) * 2.0).contiguous()
    m = 1e-4 * torch.randn(S.HEAD_PARAMS, generator=g, device=DEV)
    v = (1e-3 * (0.5 + _rand(g, S.HEAD_PARAMS))) ** 2
    return crops, stats, label, target, m, v


TRAIN_T, TRAIN_LR = 500, 1e-3


def _warp(g, size):
    """A projective sensed -> reference map about the image centre: a small
    rotation, scale, shift and perspective term (row-major 3 x 3)."""
    u = (_rand(g, 6).double() * 2 - 1).tolist()
    a, sc = math.radians(0.7 * u[0]), 1.0 + 0.004 * u[1]
    ce = 0.5 * (size - 1)
    R = np.array([[sc * math.cos(a), -sc * math.sin(a), 0], [sc * math.sin(a), sc * math.cos(a), 0], [0, 0, 1.0]])
    K = np.array([[1, 0, 0], [0, 1, 0], [2e-3 / size * u[2], 2e-3 / size * u[3], 1.0]])
    C = np.array([[1, 0, ce], [0, 1, ce], [0, 0, 1.0]])
    T = np.array([[1, 0, 5 * u[4]], [0, 1, 5 * u[5]], [0, 0, 1.0]])
    M = T @ C @ K @ R @ np.linalg.inv(C)
    return M / M[2, 2]


def _ransac_inputs(c, seed):
    """CP records of a warped scene: a third of them wrong, some at the edge
    of their window, sub-pixel noise; and the random words."""
    g = _gen(seed)
    n, size = c["n"], c["size"]
    M = torch.from_numpy(_warp(g, size)).to(DEV)
    p = torch.floor(_rand(g, n, 2).double() * (size - 200)) + 100
    h = torch.cat([p, torch.ones(n, 1, dtype=torch.float64, device=DEV)], 1) @ M.T
    d = h[:, :2] / h[:, 2:] - p + 0.3 * torch.randn(n, 2, generator=g, device=DEV)
    wrong = _rand(g, n) < 0.33
    d = torch.where(wrong[:, None], (_rand(g, n, 2).double() - 0.5) * 96.0, d)
    i = torch.round(d)
    cps = torch.zeros(n, 8, dtype=torch.int32, device=DEV)
    cps[:, :2] = p.to(torch.int32)
    cps[:, 2:4] = i.to(torch.int32)
    f = cps.view(torch.float32)
    f[:, 4:6] = (d - i).float()
    f[:, 6] = 0.2 + 0.6 * _rand(g, n)
    cps[:, 7] = torch.where(_rand(g, n) < 0.04, S.EDGE_PEAK, torch.where(wrong, S.INCONSISTENT, S.VALID)).to(torch.int32)
    k = 4 if c["model"] == "projective" else 3
    words = torch.randint(-(1 << 31), 1 << 31, (c["n_hyp"] * k,), generator=g, device=DEV, dtype=torch.int64).to(torch.int32)
    return cps, words


def _rectify_inputs(c, seed):
    g = _gen(seed)
    Hs, Ws = c["Hs"], c["Ws"]
    buf = _rand(g, Hs, Ws + c["pad"])
    sen = _field(g, Hs, Ws + c["pad"], 9).add_(0.1 * buf)[:, :Ws]
    model = torch.from_numpy(_warp(g, max(Hs, Ws)).reshape(9)).to(DEV)
    return sen, model


def _fast_inputs(c, seed):
    g = _gen(seed)
    return _images(g, 8, 8, c["H"], c["W"], 4.0, 0)[1]


# ---- the work --------------------------------------------------------------
def prepare(case, seed):
    c, k = case, case["kind"]
    if k == "pair":
        ref, sen, ips, prior = _pair_inputs(c, seed)
        p = S.preset(c["preset"], DTYPES[c["dtype"]][0])
        R = S.Registrar(c["Hr"], c["Wr"], c["Hs"], c["Ws"], c["n"], c["m"], c["r"], p, want_ncc=c["ncc"])
        return dict(kind=k, R=R, ref=ref, sen=sen, ips=ips, prior=prior)
    if k == "describe":
        img = _images(_gen(seed), c["H"], c["W"], 8, 8, 1.0, 0)[0]
        return dict(kind=k, img=img, p=S.preset(c["preset"], DTYPES[c["dtype"]][0]))
    if k == "match":
        dref, dsen, ips = _match_inputs(c, seed)
        i1, i2 = (None, None) if c["window"] else _integrals(dref)
        return dict(kind=k, dref=dref, dsen=dsen, i1=i1, i2=i2, ips=ips, m=c["m"], r=c["r"])
    if k == "plan":
        pairs = [dict(ref=a, sen=b, ips=i, m=s["m"], r=s["r"]) for s, a, b, i, _ in _plan_inputs(c, seed)]
        return dict(kind=k, plan=S.Plan(pairs, S.preset("baseline", DTYPES[c["dtype"]][0]), S.PLAN_GRAPH))
    if k == "head_train":
        crops, stats, label, target, m, v = _head_batch(c, seed)
        head = S.Head(_head_params(), device=DEV)
        head.m, head.v, head.t = m, v, TRAIN_T
        return dict(kind=k, head=head, batch=(crops, stats, label, target))
    if k == "head_infer":
        dref, dsen, ips = _match_inputs(c, seed)
        i1, i2 = _integrals(dref)
        ncc, _ = _surfaces64(dref, dsen, ips, None, c["m"], c["r"])
        ncc = ncc.float().contiguous()
        cps = _records(ncc, ips, c["r"])
        return dict(kind=k, head=S.Head(_head_params(), device=DEV), args=(dsen, dref, i1, i2, ips, c["m"], c["r"], ncc),
                    cps=cps)
    if k == "ransac":
        cps, words = _ransac_inputs(c, seed)
        model = S.MODEL_PROJECTIVE if c["model"] == "projective" else S.MODEL_AFFINE
        rp = S.ransac_params(model, c["n_hyp"], (c["size"],) * 4, 1.5, c["n_refine"])
        return dict(kind=k, R=S.Ransac(c["n"], rp), cps=cps, words=words)
    if k == "rectify":
        sen, model = _rectify_inputs(c, seed)
        out = torch.empty(c["Ho"], c["Wo"], device=DEV)
        return dict(kind=k, sen=sen, model=model, out=out, shape=(c["Ho"], c["Wo"]))
    img = _fast_inputs(c, seed)
    return dict(kind=k, D=S.Detector(c["H"], c["W"], c["nby"], c["nbx"], c["per"], c["threshold"], c["margin"]), img=img)


def _fields(cps):
    """The fields of CP records (n, 8) int32, as views."""
    f = cps.view(torch.float32)
    return dict(peak=cps[:, :4], sub=f[:, 4:6], score=f[:, 6], flags=cps[:, 7])


def run(state):
    k = state["kind"]
    if k == "pair":
        R = state["R"]
        out = _fields(R(state["ref"], state["sen"], state["ips"], state["prior"]))
        return dict(out, ncc=R.ncc) if R.ncc is not None else out
    if k == "describe":
        d, i1, i2 = S.describe(state["img"], state["p"])
        return dict(desc=d, integ1=i1, integ2=i2)
    if k == "match":
        cps, ncc = S.fastncc_match(state["dsen"], state["dref"], state["i1"], state["i2"], state["ips"], state["m"],
                                   state["r"], want_ncc=True)
        return dict(_fields(cps), ncc=ncc)
    if k == "plan":
        return [_fields(c) for c in state["plan"]()]
    if k == "head_train":
        head = state["head"]
        loss, grad = head.train_step(*state["batch"], TRAIN_LR, want_grad=True)
        return dict(loss=loss, grad=grad, params=head.params, m=head.m, v=head.v)
    if k == "head_infer":
        head, cps = state["head"], state["cps"]
        crops, stats = S.head_features(*state["args"], cps)
        out = head.infer(crops, stats, cps, want_out=True)
        return dict(_fields(cps), crops=crops, stats=stats, out=out)
    if k == "ransac":
        model, info = state["R"](state["cps"], state["words"])
        return dict(model=model, info=info, flags=state["cps"][:, 7])
    if k == "rectify":
        return S.rectify(state["sen"], state["model"], state["shape"], out=state["out"])
    ips, scores, counts, n_out = state["D"](state["img"])
    return dict(ips=ips, scores=scores, counts=counts, n_out=n_out)


# ---- what a pass cannot do without ------------------------------------------
def _sfoc_flops(preset):
    """Multiply-adds of the filter bank per pixel, as flops (separable
    passes, steering, separable smoothing per rate, normalisation)."""
    N, s1, s2 = BANK[preset]
    f = sum(8 * (2 * math.ceil(3 * s - 1e-9) + 1) for s in set(s1) & set(s2))
    f += sum(5 * (2 * math.ceil(3 * s - 1e-9) + 1) for s in set(s1) ^ set(s2))
    return 2.0 * (f + 5 * N + 2 * N * 3 * 6 + 4 * N + 2)


def _match_flops(n, m, r, z):
    M, V = m + 2 * r, 2 * r + 1
    return n * ((2 * z + 1) * 2.5 * M * M * 2 * math.log2(M) + 8.0 * z * M * (M / 2 + 1) + 20.0 * V * V)


def _pair_work(c):
    N = BANK[c["preset"]][0]
    M = c["m"] + 2 * c["r"]
    nr, ns = c["Hr"] * c["Wr"], c["Hs"] * c["Ws"]
    px = min(nr, c["n"] * M * M) + min(ns, c["n"] * c["m"] ** 2)
    V = 2 * c["r"] + 1
    return (4.0 * px + 40.0 * c["n"] + (4.0 * c["n"] * V * V if c.get("ncc") else 0),
            px * _sfoc_flops(c["preset"]) + _match_flops(c["n"], c["m"], c["r"], 2 * N))


def work(case):
    c, k = case, case["kind"]
    if k == "pair":
        b, f = _pair_work(c)
    elif k == "describe":
        px, N = c["H"] * c["W"], BANK[c["preset"]][0]
        b, f = px * (4.0 + 2 * N * ES[c["dtype"]] + 16.0), px * _sfoc_flops(c["preset"])
    elif k == "match":
        px, M, V, e = c["H"] * c["W"], c["m"] + 2 * c["r"], 2 * c["r"] + 1, ES[c["dtype"]]
        b = 16.0 * e * (min(px, c["n"] * M * M) + min(px, c["n"] * c["m"] ** 2)) + c["n"] * (40.0 + 4.0 * V * V)
        b += 0 if c["window"] else 16.0 * min(px, 4 * c["n"] * V * V)
        f = _match_flops(c["n"], c["m"], c["r"], 16)
    elif k == "plan":
        w = [_pair_work(s) for s in _plan_specs(c)]
        b, f = sum(x[0] for x in w), sum(x[1] for x in w)
    elif k == "head_train":
        b, f = c["n"] * (33 * 33 + 8 + 3) * 4.0 + 7 * 4.0 * S.HEAD_PARAMS, 3.0 * _net_flops(c["n"])
    elif k == "head_infer":
        V = 2 * c["r"] + 1
        b = c["n"] * (4.0 * V * V + 2 * 4.0 * (33 * 33 + 8) + 16.0 * c["m"] ** 2 * ES[c["dtype"]] + 64 + 64)
        f = _net_flops(c["n"]) + c["n"] * (4.0 * V * V + 48.0 * c["m"] ** 2)
    elif k == "ransac":
        t = 21 if c["model"] == "projective" else 13
        b, f = c["n"] * 36.0 + c["n_hyp"] * 16.0, float(t) * c["n"] * c["n_hyp"]
    elif k == "rectify":
        b, f = 4.0 * (min(c["Hs"] * c["Ws"], c["Ho"] * c["Wo"]) + c["Ho"] * c["Wo"]), 25.0 * c["Ho"] * c["Wo"]
    else:
        b, f = 4.0 * c["H"] * c["W"], 82.0 * c["H"] * c["W"]
    return {"bytes": b, "flops": f}


def _net_flops(n):
    return 2.0 * n * (33 * 33 * 9 * 32 + (17 * 17 + 81 + 25) * 9 * 32 * 32 + 808 * 32 + 96)


# ---- the same in 64 bits ----------------------------------------------------
def _sfoc64(img, preset):
    """Dense descriptor (z, H, W) in float64: basis responses on the
    reflect-101 extended image summed over scales, steered, rectified,
    smoothed at three rates, normalised per order."""
    N, s1, s2 = BANK[preset]
    R = max(math.ceil(3 * s - 1e-9) for s in s1 + s2)
    P = R + Q
    H, W = img.shape

    def mirror(n):
        i = torch.arange(-P, n + P, device=DEV) % max(1, 2 * (n - 1))
        return torch.where(i > n - 1, 2 * (n - 1) - i, i)

    E = img.double()[mirror(H)][:, mirror(W)]
    H2, W2 = H + 2 * Q, W + 2 * Q

    def taps(s, kind):
        rad = math.ceil(3 * s - 1e-9)
        k = np.arange(-rad, rad + 1, dtype=np.float64)
        e = np.exp(-k * k / (2 * s * s))
        return {"g": e, "d": -k / (s * s) * e, "dd": (k * k / s ** 4 - 1 / (s * s)) * e}[kind], rad

    def conv(x, s, kind, axis, n):
        """Convolution along an axis, to the n positions the Q border leaves."""
        t, rad = taps(s, kind)
        out = None
        o = (x.shape[axis] - n) // 2
        for j, w in enumerate(t):
            y = x.narrow(axis, o + rad - j, n) * w       # out[p] = sum_k t[k] x[p - k], k = j - rad
            out = y if out is None else out.add_(y)
        return out

    zero = [None] * 5

    def add(i, v, w):
        zero[i] = v * w if zero[i] is None else zero[i].add_(v, alpha=w)

    for s in sorted(set(s1) | set(s2)):
        cn = 1.0 / (2 * math.pi * s * s)
        g, d = conv(E, s, "g", 1, W2), conv(E, s, "d", 1, W2)
        if s in s1:
            add(0, conv(d, s, "g", 0, H2), cn)
            add(1, conv(g, s, "d", 0, H2), cn)
        if s in s2:
            dd = conv(E, s, "dd", 1, W2)
            add(2, conv(dd, s, "g", 0, H2), cn)
            add(3, conv(g, s, "dd", 0, H2), cn)
            add(4, conv(d, s, "d", 0, H2), cn)
            del dd
        del g, d
    bx, by, bxx, byy, bxy = zero
    out = torch.empty(2 * N, H, W, dtype=torch.float64, device=DEV)
    for o in range(2):
        w = np.exp(-np.arange(-1, 2) ** 2 / (2.0 * (SD2 if o else SD1) ** 2))
        w = w / w.sum()
        for i in range(N):
            c, sn = math.cos(i * math.pi / N), math.sin(i * math.pi / N)
            a = (c * c * bxx + sn * sn * byy + 2 * sn * c * bxy if o else c * bx + sn * by).abs_()
            acc = out[o * N + i].zero_()
            for rt in RATES:
                v = sum(w[j] * a.narrow(0, Q + (j - 1) * rt, H) for j in range(3))
                for j in range(3):
                    acc.add_(v.narrow(1, Q + (j - 1) * rt, W), alpha=float(w[j]))
        blk = out[o * N:(o + 1) * N]
        norm = torch.zeros(H, W, dtype=torch.float64, device=DEV)
        for ch in blk:
            norm.addcmul_(ch, ch)
        norm.add_(EPS).sqrt_()
        for ch in blk:
            ch.div_(norm)
    return out


def _surfaces64(dref, dsen, ips, prior, m, r):
    """NCC surfaces (n, V, V) in float64 for descriptors (z, H, W), and their
    maxima."""
    z, n, M, V = dref.shape[0], ips.shape[0], m + 2 * r, 2 * r + 1
    L = -(-M // 32) * 32
    mnz = float(m * m * z)
    out = torch.empty(n, V, V, dtype=torch.float64, device=DEV)
    i64 = ips.long()
    ty, tx = i64[:, 0] - m // 2, i64[:, 1] - m // 2
    sy, sx = ty - r, tx - r
    if prior is not None:
        sy, sx = sy + prior[:, 0].long(), sx + prior[:, 1].long()
    am, aM = torch.arange(m, device=DEV), torch.arange(M, device=DEV)
    step = max(1, min(n, (1 << 26) // (z * L * L)))
    for b in range(0, n, step):
        e = min(n, b + step)

        def window(d, y, x, a):
            return d[:, (y[b:e, None] + a)[:, :, None], (x[b:e, None] + a)[:, None, :]].double()

        T, W = window(dsen, ty, tx, am), window(dref, sy, sx, aM)
        F = torch.fft.rfft2(W, s=(L, L))
        F.mul_(torch.fft.rfft2(T, s=(L, L)).conj())
        RST = torch.fft.irfft2(F.sum(0), s=(L, L))[:, :V, :V]
        RT, RTT = T.sum((0, 2, 3)), (T * T).sum((0, 2, 3))
        box = []
        for g in (W.sum(0), (W * W).sum(0)):
            I = torch.zeros(e - b, M + 1, M + 1, dtype=torch.float64, device=DEV)
            I[:, 1:, 1:] = g.cumsum(1).cumsum(2)
            box.append(I[:, m:, m:] - I[:, :V, m:] - I[:, m:, :V] + I[:, :V, :V])
        varT = (RTT - RT * RT / mnz)[:, None, None]
        varS = box[1] - box[0] * box[0] / mnz
        tau = 1e-12 * mnz
        val = (RST - box[0] * RT[:, None, None] / mnz) / torch.sqrt((varS * varT).clamp_min(1e-300))
        out[b:e] = torch.where((varS > tau) & (varT > tau), val, torch.zeros_like(val))
    return out, out.flatten(1).max(1).values


def _records(ncc, ips, r):
    """CP records of surfaces: integer peak, parabola, VALID (or EDGE_PEAK)."""
    n, V = ncc.shape[0], 2 * r + 1
    best, at = ncc.flatten(1).max(1)
    u, v = at // V, at % V
    inner = (u > 0) & (u < V - 1) & (v > 0) & (v < V - 1)
    row = torch.arange(n, device=DEV)
    cps = torch.zeros(n, 8, dtype=torch.int32, device=DEV)
    cps[:, :2] = ips
    cps[:, 2], cps[:, 3] = (u - r).int(), (v - r).int()
    f = cps.view(torch.float32)
    uc, vc = u.clamp(1, V - 2), v.clamp(1, V - 2)
    for col, (a, b) in ((4, ((uc - 1, vc), (uc + 1, vc))), (5, ((uc, vc - 1), (uc, vc + 1)))):
        lo, hi = ncc[row, a[0], a[1]], ncc[row, b[0], b[1]]
        den = lo - 2 * best + hi
        d = torch.where(den < 0, (lo - hi) / (2 * den), torch.zeros_like(den)).clamp(-0.5, 0.5)
        f[:, col] = torch.where(inner, d, torch.zeros_like(d))
    f[:, 6] = best
    cps[:, 7] = torch.where(inner, S.VALID, S.EDGE_PEAK).to(torch.int32)
    return cps


def _bf16(x):
    return x.to(torch.bfloat16).double()


def _net64(theta, crops, stats):
    """The head in float64: weights rounded to bfloat16, biases as they are.
    Returns (out, the 12 parameter leaves as the network reads them)."""
    leaves, o = [], 0
    for s in HEAD_SHAPES:
        k = int(np.prod(s))
        t = theta[o:o + k].reshape(s)
        leaves.append((_bf16(t) if len(s) > 1 else t.double()).requires_grad_(True))
        o += k
    x = crops.double()[:, None]
    for i in range(4):
        x = torch.relu(torch.nn.functional.conv2d(x, leaves[2 * i], leaves[2 * i + 1], stride=1 if i == 0 else 2, padding=1))
    x = torch.cat([x.flatten(1), stats.double()], 1)
    x = torch.relu(x @ leaves[8].T + leaves[9])
    return x @ leaves[10].T + leaves[11], leaves


def exact(case, seed):
    c, k = case, case["kind"]
    if k == "pair":
        ref, sen, ips, prior = _pair_inputs(c, seed)
        ncc, best = _surfaces64(_sfoc64(ref, c["preset"]), _sfoc64(sen, c["preset"]), ips, prior, c["m"], c["r"])
        out = dict(peak=None, sub=None, score=best, flags=None)
        return dict(out, ncc=ncc) if c["ncc"] else out
    if k == "describe":
        d = _sfoc64(_images(_gen(seed), c["H"], c["W"], 8, 8, 1.0, 0)[0], c["preset"])
        i1, i2 = _integrals(d)
        return dict(desc=d, integ1=i1, integ2=i2)
    if k == "match":
        dref, dsen, ips = _match_inputs(c, seed)
        ncc, best = _surfaces64(dref, dsen, ips, None, c["m"], c["r"])
        return dict(peak=None, sub=None, score=best, flags=None, ncc=ncc)
    if k == "plan":
        out = []
        for s, ref, sen, ips, prior in _plan_inputs(c, seed):
            best = _surfaces64(_sfoc64(ref, "baseline"), _sfoc64(sen, "baseline"), ips, prior, s["m"], s["r"])[1]
            out.append(dict(peak=None, sub=None, score=best, flags=None))
        return out
    if k == "head_train":
        return _train64(c, seed)
    if k == "head_infer":
        return _infer64(c, seed)
    if k == "ransac":
        cps, words = _ransac_inputs(c, seed)
        return dict(model=_ransac64(c, cps, words), info=None, flags=None)
    if k == "rectify":
        return _rectify64(c, seed)
    return _fast64(c, seed)


def _train64(c, seed):
    crops, stats, label, target, m, v = (t.cpu() for t in _head_batch(c, seed))
    theta = _head_params()
    out, leaves = _net64(theta, crops, stats)
    y = label.double()
    l1 = torch.nn.functional.smooth_l1_loss(out[:, 1:], target.double(), beta=0.1, reduction="none").sum(1)
    loss = (torch.nn.functional.binary_cross_entropy_with_logits(out[:, 0], y, reduction="none") + 4 * y * l1).mean()
    g = torch.cat([t.flatten() for t in torch.autograd.grad(loss, leaves)])
    t = TRAIN_T + 1
    m2 = 0.9 * m.double() + 0.1 * g
    v2 = 0.999 * v.double() + 0.001 * g * g
    p = theta.double() - TRAIN_LR * (m2 / (1 - 0.9 ** t)) / (torch.sqrt(v2 / (1 - 0.999 ** t)) + 1e-8)
    return dict(loss=loss.detach().reshape(1), grad=g, params=p, m=m2, v=v2)


def _infer64(c, seed):
    dref, dsen, ips = _match_inputs(c, seed)
    m, r = c["m"], c["r"]
    ncc = _surfaces64(dref, dsen, ips, None, m, r)[0].float()
    cps = _records(ncc, ips, r)
    n, V, z = c["n"], 2 * r + 1, dref.shape[0]
    S64 = ncc.double()
    u, v = (cps[:, 2] + r).long(), (cps[:, 3] + r).long()
    keep = cps[:, 7] == S.VALID
    pad = torch.full((n, V + 32, V + 32), -1.0, dtype=torch.float64, device=DEV)
    pad[:, 16:-16, 16:-16] = S64
    row, a33 = torch.arange(n, device=DEV), torch.arange(33, device=DEV)
    crops = pad[row[:, None, None], (u[:, None] + a33)[:, :, None], (v[:, None] + a33)[:, None, :]]
    yy, xx = torch.arange(V, device=DEV)[None, :, None], torch.arange(V, device=DEV)[None, None, :]
    near = ((yy - u[:, None, None]).abs() <= 1) & ((xx - v[:, None, None]).abs() <= 1)
    second = torch.where(near, -1.0, S64).flatten(1).amax(1).clamp_min(-1.0)
    flat = S64.flatten(1)
    std = flat.std(1, unbiased=False)
    mnz = float(m * m * z)
    am = torch.arange(m, device=DEV)

    def box(d, y, x):
        s1, s2 = torch.zeros(n, dtype=torch.float64, device=DEV), torch.zeros(n, dtype=torch.float64, device=DEV)
        for ch in d:
            w = ch[(y[:, None] + am)[:, :, None], (x[:, None] + am)[:, None, :]].double()
            s1 += w.sum((1, 2))
            s2 += (w * w).sum((1, 2))
        return s1, s2

    ty, tx = ips[:, 0].long() - m // 2, ips[:, 1].long() - m // 2
    RT, RTT = box(dsen, ty, tx)
    uc, vc = u.clamp(1, V - 2), v.clamp(1, V - 2)
    RS, RSS = box(dref, ty - r + u, tx - r + v)
    c0 = S64[row, u, v]
    curv = 0.5 * (S64[row, uc - 1, vc] + S64[row, uc + 1, vc] + S64[row, uc, vc - 1] + S64[row, uc, vc + 1] - 4 * c0)
    stats = torch.stack([c0, second, flat.mean(1), std, torch.sqrt((RTT - RT * RT / mnz).clamp_min(0) / mnz),
                         torch.sqrt((RSS - RS * RS / mnz).clamp_min(0) / mnz), RT / mnz, curv], 1)
    crops, stats = crops * keep[:, None, None], stats * keep[:, None]
    out, _ = _net64(_head_params(), crops.cpu(), stats.cpu())
    return dict(peak=None, sub=None, score=None, flags=None, crops=crops, stats=stats, out=out.detach())


def _ransac64(c, cps, words):
    """The model of RANSAC in float64: minimal fits by linear solves, the
    first hypothesis with the most inliers, least-squares refits."""
    a = cps.cpu().numpy()
    f = a.view(np.float32)
    a, f = a[a[:, 7] != S.EDGE_PEAK], f[a[:, 7] != S.EDGE_PEAK]
    size, proj = c["size"], c["model"] == "projective"
    k, half, ctr = (4, 0.5 * size, 0.5 * (size - 1)) if proj else (3, 0.5 * size, 0.5 * (size - 1))
    src = (a[:, :2].astype(np.float64) - ctr) / half
    dst = (a[:, :2].astype(np.float64) + a[:, 2:4] + f[:, 4:6] - ctr) / half
    n = len(src)
    w = words.cpu().numpy().view(np.uint32).astype(np.uint64).reshape(-1, k)
    sel = ((w * np.uint64(n)) >> np.uint64(32)).astype(np.int64)

    def rows(s, d):
        """Linear system of the map (h22 = 1) from points s to d (.., k, 2)."""
        x, y, X, Y = s[..., 0], s[..., 1], d[..., 0], d[..., 1]
        o, z = np.ones_like(x), np.zeros_like(x)
        p = 8 if proj else 6
        r1 = np.stack([x, y, o, z, z, z, -x * X, -y * X][:p], -1)
        r2 = np.stack([z, z, z, x, y, o, -x * Y, -y * Y][:p], -1)
        return np.concatenate([r1, r2], -2), np.concatenate([X, Y], -1)

    def inside(M):
        h = src @ M[..., :2].swapaxes(-1, -2) + M[..., None, :, 2]
        den = h[..., 2]
        e = ((h[..., :2] - dst * den[..., None]) ** 2).sum(-1)
        return (den > 0) & (e <= (1.5 / half) ** 2 * den * den)

    def full(h):
        return np.concatenate([h, np.zeros(h.shape[:-1] + (8 - h.shape[-1],)), np.ones(h.shape[:-1] + (1,))], -1).reshape(h.shape[:-1] + (3, 3))

    A, b = rows(src[sel], dst[sel])
    good = np.array([len(set(q)) == k for q in sel.tolist()])
    good &= np.abs(np.linalg.det(A)) > 1e-30
    Ms = np.zeros((len(sel), 3, 3))
    Ms[good] = full(np.linalg.solve(A[good], b[good][..., None])[..., 0])
    count = np.full(len(sel), -1)
    for i in range(0, len(sel), 256):
        count[i:i + 256] = inside(Ms[i:i + 256]).sum(-1)
    count[~good] = -1
    M = Ms[int(np.argmax(count))]
    inl = inside(M)
    for _ in range(c["n_refine"]):
        A, b = rows(src[inl], dst[inl])
        M = full(np.linalg.lstsq(A, b, rcond=None)[0])
        inl = inside(M)
    Ts = np.array([[1 / half, 0, -ctr / half], [0, 1 / half, -ctr / half], [0, 0, 1.0]])
    Pm = np.linalg.inv(Ts) @ M @ Ts
    return (Pm / Pm[2, 2]).reshape(9)


def _rectify64(c, seed):
    sen, model = _rectify_inputs(c, seed)
    Mi = torch.from_numpy(np.linalg.inv(model.cpu().numpy().reshape(3, 3))).to(DEV)
    Hs, Ws, Ho, Wo = c["Hs"], c["Ws"], c["Ho"], c["Wo"]
    out = torch.empty(Ho, Wo, dtype=torch.float64, device=DEV)
    col = torch.arange(Wo, device=DEV, dtype=torch.float64)[None, :]
    for r0 in range(0, Ho, 512):
        row = torch.arange(r0, min(Ho, r0 + 512), device=DEV, dtype=torch.float64)[:, None]
        w = Mi[2, 0] * row + Mi[2, 1] * col + Mi[2, 2]
        y = (Mi[0, 0] * row + Mi[0, 1] * col + Mi[0, 2]) / w
        x = (Mi[1, 0] * row + Mi[1, 1] * col + Mi[1, 2]) / w
        ok = (w > 0) & (y >= 0) & (y <= Hs - 1) & (x >= 0) & (x <= Ws - 1)
        y, x = torch.where(ok, y, 0.0), torch.where(ok, x, 0.0)
        y0, x0 = y.floor().long(), x.floor().long()
        y1, x1 = (y0 + 1).clamp_max(Hs - 1), (x0 + 1).clamp_max(Ws - 1)
        fy, fx = y - y0, x - x0
        top = sen[y0, x0].double() * (1 - fx) + sen[y0, x1].double() * fx
        bot = sen[y1, x0].double() * (1 - fx) + sen[y1, x1].double() * fx
        out[r0:r0 + 512] = torch.where(ok, top * (1 - fy) + bot * fy, 0.0)
    return out


def _fast64(c, seed):
    """Corner strengths of the selected points (their order is the point
    order; the points themselves are whole numbers)."""
    img = _fast_inputs(c, seed).double()
    H, W, b = c["H"], c["W"], max(3, c["margin"])
    ring = [(-3, 0), (-3, 1), (-2, 2), (-1, 3), (0, 3), (1, 3), (2, 2), (3, 1), (3, 0), (3, -1), (2, -2), (1, -3),
            (0, -3), (-1, -3), (-2, -2), (-3, -1)]
    h, w = H - 2 * b, W - 2 * b
    V = torch.full((H, W), -math.inf, dtype=torch.float64, device=DEV)
    for r0 in range(0, h, 1024):
        e = min(h, r0 + 1024)
        at = [img[b + r0 + dy:b + e + dy, b + dx:b + dx + w] for dy, dx in ring]
        ctr = img[b + r0:b + e, b:b + w]
        best = torch.full_like(ctr, -math.inf)
        for q in range(16):
            lo, hi = at[q].clone(), at[q].clone()
            for j in range(1, 9):
                torch.minimum(lo, at[(q + j) % 16], out=lo)
                torch.maximum(hi, at[(q + j) % 16], out=hi)
            best = torch.maximum(best, torch.maximum(lo - ctr, ctr - hi))
        V[b + r0:b + e, b:b + w] = best
    keep = V > c["threshold"]
    keep[0], keep[-1], keep[:, 0], keep[:, -1] = False, False, False, False
    mid = V[1:-1, 1:-1]
    for dy, dx in ((-1, -1), (-1, 0), (-1, 1), (0, -1), (0, 1), (1, -1), (1, 0), (1, 1)):
        o = V[1 + dy:H - 1 + dy, 1 + dx:W - 1 + dx]
        keep[1:-1, 1:-1] &= (mid > o) if (dy, dx) < (0, 0) else (mid >= o)
    yx = keep.nonzero().cpu().numpy()
    s = V[keep].cpu().numpy()
    ey = b + np.arange(c["nby"] + 1) * h // c["nby"]
    ex = b + np.arange(c["nbx"] + 1) * w // c["nbx"]
    blk = (np.searchsorted(ey, yx[:, 0], "right") - 1) * c["nbx"] + np.searchsorted(ex, yx[:, 1], "right") - 1
    order = np.lexsort((np.arange(len(s)), -s, blk))
    blk, s = blk[order], s[order]
    first = np.searchsorted(blk, blk, "left")
    s = s[np.arange(len(s)) - first < c["per"]]
    scores = np.zeros(c["nby"] * c["nbx"] * c["per"])
    scores[:len(s)] = s
    return dict(ips=None, scores=scores, counts=None, n_out=None)
