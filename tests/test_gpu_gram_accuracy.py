"""The Gram kernel's rounding where resident waves share rows evenly: against exact integer sums, no larger
than with every item in the scratch's parts (a point at a time), whose chains of sums are short.  The
matrix cores' sums of like sign drift in proportion to a chain's length."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n,nv,ntb,nseg", [(40013, 80, 125, 9), (40013, 44, 125, 9), (45001, 64, 70, 9),
                                           (40013, 96, 60, 9), (40013, 128, 40, 9)])
def test_gram_shares_round_like_parts(precision, n, nv, ntb, nseg):
    from paper_1504_07690_amd import ssm as S
    dt = torch.float64 if precision == "fp64" else torch.float32
    g = torch.Generator(device=DEV).manual_seed(n + nv)
    # integers of 23 bits: products below 2^46, sums below 2^62, exact in int64
    w = torch.randint(1 << 22, 1 << 23, (n, nv), device=DEV, generator=g).to(dt)
    z = torch.empty(ntb, n, nv, dtype=dt, device=DEV)
    for i in range(ntb):
        z[i] = torch.randint(1 << 22, 1 << 23, (n, nv), device=DEV, generator=g).to(dt)
    kw = torch.empty(ntb, nv, nv, dtype=torch.float64, device=DEV)
    kz = torch.empty_like(kw)
    S.gram(precision, w, z, kw, kz, nseg=nseg)
    k1, k2 = torch.empty(1, nv, nv, dtype=torch.float64, device=DEV), torch.empty(1, nv, nv, dtype=torch.float64,
                                                                                  device=DEV)
    err = {}
    cols = min(nv, 16)  # the first block row of Z^T Z, in which every entry is stored as formed but the first block
    for i in (0, ntb // 2, ntb - 1):
        S.gram(precision, w, z[i: i + 1], k1, k2, nseg=nseg)
        zi = z[i].cpu().numpy().astype(np.int64)
        exact = zi[:, :cols].T @ zi
        for name, k in (("shares", kz[i]), ("parts", k2[0])):
            d = k.cpu().numpy()[:cols].astype(np.int64) - exact
            err.setdefault(name, []).append((d.astype(np.float64) / exact) ** 2)
    rms = {name: float(np.sqrt(np.mean(e))) for name, e in err.items()}
    # chains no longer than the parts': the same error up to what the rounding of three points scatters
    assert rms["shares"] <= 1.5 * rms["parts"], rms
