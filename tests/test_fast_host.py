"""The FAST workspace's queried size is a strength per pixel and a mask word per 32
pixels of a row beside the blocks' records, at every image size: a size that a
caller has stored stays enough."""
import pytest

from paper_2202_13347_amd import sfoc as S


def stored(H, W, nby, nbx, per):
    up = lambda b: (max(b, 1) + 255) // 256 * 256
    k = nby * nbx * per
    return up(4 * H * W) + up(4 * H * ((W + 31) // 32)) + up(8 * k) + up(4 * k) + up(4 * nby * nbx)


@pytest.mark.parametrize("nby,nbx,per", [(1, 1, 1), (71, 71, 1), (3, 5, 32)])
def test_workspace_size(nby, nbx, per):
    for H in (1, 6, 7, 8, 31, 32, 33, 100, 1000, 1 << 20):
        for W in (1, 2, 6, 7, 8, 9, 31, 32, 33, 65, 1000, 4096):
            assert S.fast_workspace(H, W, nby, nbx, per) == stored(H, W, nby, nbx, per), (H, W)
