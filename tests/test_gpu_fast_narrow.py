"""FAST on narrow and small images, their lists as full as suppression allows, in
a workspace of exactly the queried size: the oracle's points, and nothing written
past it."""
import ctypes

import numpy as np
import pytest

from oracle import fast_oracle as F
from paper_2202_13347_amd import sfoc as S

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("H,W,nby,nbx,per", [(1000, 8, 5, 1, 32), (8, 1000, 1, 7, 32), (7, 7, 1, 1, 2), (500, 7, 9, 1, 8),
                                             (7, 500, 1, 9, 8), (65, 39, 2, 2, 32), (6, 300, 1, 2, 4), (300, 5, 2, 1, 4),
                                             (1, 1, 1, 1, 1)])
def test_exact_workspace(H, W, nby, nbx, per):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print("fast narrow", H, W, nby, nbx, per, flush=True)
    img = np.zeros((H, W), np.float32)
    img[::2, ::2] = 1 + np.random.default_rng(H + W).random(img[::2, ::2].shape)
    dev = torch.from_numpy(img).cuda()
    up = lambda b: (max(b, 1) + 255) // 256 * 256
    cap = nby * nbx * per
    size = up(4 * H * W) + up(4 * H * ((W + 31) // 32)) + up(8 * cap) + up(4 * cap) + up(4 * nby * nbx)
    ws = torch.full((size + 4096,), 0x5a, dtype=torch.uint8, device="cuda")
    ips, sc = torch.full((cap, 2), -1, dtype=torch.int32, device="cuda"), torch.zeros(cap, device="cuda")
    cnt, n = (torch.full((k,), -1, dtype=torch.int32, device="cuda") for k in (nby * nbx, 1))
    call = lambda b: S.lib().sfoc_detect_ips(S._ptr(dev), H, W, W, ctypes.c_float(0.0), 0, nby, nbx, per, S._ptr(ips),
                                             S._ptr(sc), S._ptr(cnt), S._ptr(n), S._ptr(ws), b, S._stream(None))
    assert call(size) == S.SFOC_OK
    torch.cuda.synchronize()
    o_ips, o_sc, o_cnt = F.detect(img, 0.0, 0, nby, nbx, per)
    k = int(n)
    assert k == len(o_ips) and np.array_equal(cnt.cpu().numpy(), np.asarray(o_cnt).reshape(-1))
    assert np.array_equal(ips[:k].cpu().numpy(), np.asarray(o_ips).reshape(-1, 2)) and np.array_equal(sc[:k].cpu().numpy(), o_sc)
    assert bool((ws[size:] == 0x5a).all())
    assert call(size - 1) == S.SFOC_E_WORKSPACE
