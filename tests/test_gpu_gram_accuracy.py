"""The Gram kernel's rounding where resident waves share rows evenly: against compensated sums, no larger than
with every item in the scratch's parts (a point at a time), whose chains of sums are short."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _gram(a):
    """a^T a as hi + lo: sums of 16 rows, added pairwise with their rounding errors kept (two-sum)."""
    n, nv = a.shape
    m = n // 16 * 16
    b = a[:m].view(-1, 16, nv)
    s = torch.bmm(b.transpose(1, 2).contiguous(), b.contiguous())
    s = torch.cat([s, (a[m:].T.contiguous() @ a[m:])[None]])
    lo = torch.zeros_like(s)
    while s.shape[0] > 1:
        if s.shape[0] % 2:
            s, lo = torch.cat([s, torch.zeros_like(s[:1])]), torch.cat([lo, torch.zeros_like(lo[:1])])
        x, y = s[0::2], s[1::2]
        s = x + y
        bb = s - x
        lo = lo[0::2] + lo[1::2] + ((x - (s - bb)) + (y - bb))
    return s[0], lo[0]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n,nv,ntb,nseg", [(40013, 80, 125, 9), (40013, 44, 125, 9), (45001, 64, 70, 9),
                                           (40013, 96, 60, 9), (40013, 128, 40, 9)])
def test_gram_shares_round_like_parts(precision, n, nv, ntb, nseg):
    from paper_1504_07690_amd import ssm as S
    dt = torch.float64 if precision == "fp64" else torch.float32
    g = torch.Generator(device=DEV).manual_seed(n + nv)
    w = torch.randn(n, nv, dtype=dt, device=DEV, generator=g)
    z = torch.empty(ntb, n, nv, dtype=dt, device=DEV)
    for i in range(ntb):
        z[i] = torch.randn(n, nv, dtype=dt, device=DEV, generator=g)
    kw = torch.empty(ntb, nv, nv, dtype=torch.float64, device=DEV)
    kz = torch.empty_like(kw)
    S.gram(precision, w, z, kw, kz, nseg=nseg)
    one_w, one_z = torch.empty_like(kw[:1]), torch.empty_like(kz[:1])
    shares, parts = [], []
    for i in (0, ntb // 2, ntb - 1):
        S.gram(precision, w, z[i: i + 1], one_w, one_z, nseg=nseg)
        hi, lo = _gram(z[i].double())
        for k, err in ((kz[i], shares), (one_z[0], parts)):
            err.append(((((k - hi) - lo).diagonal() / hi.diagonal()) ** 2).mean().item())
    # chains no longer than the parts': the same error up to what the rounding of three points scatters
    assert np.sqrt(np.mean(shares)) <= 1.5 * np.sqrt(np.mean(parts)), (shares, parts)
