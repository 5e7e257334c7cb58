"""Fast-NCC surfaces at the extents where the match kernels change form.

Transforms: windows and templates that end at, just before and just after half
and three quarters of each transform side (the samples beyond them are not
read), odd sides (a row pair with one row missing), and the smallest and
largest of each side."""
import numpy as np
import pytest

from oracle import sfoc_oracle as O
from paper_2202_13347_amd import sfoc as S
from paper_2202_13347_amd import synth
from tests.gpu_util import compare_cps, to_chw

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def check_surface(m, r, dt):
    """Surfaces and records of windows that touch the image borders against
    the oracle on the same (rounded) descriptors, integral images per window."""
    print("extents", m, r, dt, flush=True)
    size = m + 2 * r + 9
    pr = synth.make_pair(500 + m + r, size, min(6.0, max(0.5, r - 2.0)))
    lo, hi = m // 2 + r, size - (m - m // 2) - r
    ips = np.array([[lo, lo], [hi, hi], [(lo + hi) // 2, hi], [hi, lo]], np.int32)   # windows on the borders
    Fs, Fr = (torch.from_numpy(np.ascontiguousarray(to_chw(O.sfoc(x)), np.float32)).to(DTYPES[dt])
              for x in (pr.sen, pr.ref))
    o, so = O.match(Fs.double().numpy().transpose(1, 2, 0), Fr.double().numpy().transpose(1, 2, 0), ips, m, r,
                    want_surfaces=True)
    cps, ncc = S.fastncc_match(Fs.cuda(), Fr.cuda(), None, None, torch.from_numpy(ips).cuda(), m, r, want_ncc=True)
    torch.cuda.synchronize()
    st = compare_cps(S.cps_to_numpy(cps), o, so, r, ncc.cpu().numpy(), check_consistency=False)
    assert st["compared"] > 0


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("m", [3, 4, 5])
def test_direct_form_smallest_templates(m, dt):
    """The direct form deals template rows to four waves; a template of three
    rows leaves the fourth none."""
    check_surface(m, 2, dt)


# (m, r): windows of side m + 2r
EXTENTS = [(3, 1), (31, 8), (32, 8), (33, 8), (32, 16), (48, 8), (49, 7),        # side 64
           (63, 1), (64, 16), (65, 16), (96, 16), (97, 15), (64, 32),            # side 128
           (79, 40), (80, 40), (81, 39), (120, 20), (121, 19), (64, 48),         # side 160
           (95, 48), (96, 48), (97, 47), (144, 24), (145, 23), (20, 86)]         # side 192


@pytest.mark.parametrize("dt", list(DTYPES))
@pytest.mark.parametrize("m,r", EXTENTS)
def test_surface_at_transform_extents(m, r, dt):
    check_surface(m, r, dt)


@pytest.mark.parametrize("m,r", [(5, 30), (9, 92), (100, 100), (30, 300)])
def test_window_integrals_at_wide_windows(m, r):
    """Integral images per window at one, several and many bands of rows and
    more columns than a wave, against those of the whole reference image."""
    print("window integrals", m, r, flush=True)
    g = torch.Generator().manual_seed(m + r)
    size = m + 2 * r + 5
    d = torch.rand(6, size, size, generator=g).cuda()
    s = torch.rand(6, size, size, generator=g).cuda()
    lo = m // 2 + r
    ips = torch.tensor([[lo, lo], [lo + 3, lo + 5]], dtype=torch.int32).cuda()
    I = []
    for k in (1, 2):
        i = torch.zeros(size + 1, size + 1, dtype=torch.float64, device="cuda")
        i[1:, 1:] = (d.double() ** k).sum(0).cumsum(0).cumsum(1)
        I.append(i)
    cw, nw = S.fastncc_match(s, d, None, None, ips, m, r, want_ncc=True)
    cg, ng = S.fastncc_match(s, d, I[0], I[1], ips, m, r, want_ncc=True)
    torch.cuda.synchronize()
    # the box sums differ by float64 rounding of sums of up to 6 size^2 values (relative 1e-12),
    # the variances (their difference, at least 1e-3 of the sums here) by 1e-9 at most
    assert float((nw - ng).abs().max()) <= 1e-6
    assert torch.equal(cw[:, :4], cg[:, :4])
