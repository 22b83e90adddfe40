"""The Gram kernel's split of rows over waves: equal shares that cross points and tiles, every item in
parts, row counts that no unit of rows divides, every tile size, scratch of one segment."""

import pytest
import torch


pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n,nv,ntb,nseg", [
    (1, 4, 1, 1), (7, 12, 3, 1), (9, 16, 2, 3), (65, 20, 5, 2), (255, 40, 4, 64), (1003, 72, 3, 1),   # in parts
    (1777, 8, 300, 8), (1700, 20, 200, 7), (4999, 40, 40, 20), (4101, 64, 33, 16), (4001, 68, 17, 16),  # shares
    (4003, 92, 17, 16), (4903, 100, 6, 20), (4903, 128, 6, 20), (5001, 132, 3, 33), (2603, 256, 3, 11),
    (5003, 128, 6, 16), (300, 200, 2, 1)])
def test_gram_every_split(precision, n, nv, ntb, nseg):
    from paper_1504_07690_amd import ssm as S
    dt = torch.float64 if precision == "fp64" else torch.float32
    g = torch.Generator(device=DEV).manual_seed(n + nv)
    w = torch.randn(n, nv, dtype=dt, device=DEV, generator=g)
    z = torch.randn(ntb, n, nv, dtype=dt, device=DEV, generator=g)
    kw = torch.full((ntb, nv, nv), float("nan"), dtype=torch.float64, device=DEV)
    kz = torch.full_like(kw, float("nan"))
    S.gram(precision, w, z, kw, kz, nseg=nseg)
    blk = torch.arange(nv, device=DEV) // 16
    upper, same = blk[:, None] < blk[None, :], blk[:, None] == blk[None, :]
    wd = w.double()
    for i in range(ntb):
        zi = z[i].double()
        m = wd.T @ zi
        ref_w = torch.where(upper, m, torch.where(same, 0.5 * (m + m.T), m.T))
        # n products summed in any order on both sides
        bw = 2 * n * 2.0 ** -53 * (wd.abs().T @ zi.abs())
        bw = torch.maximum(bw, bw.T)
        bz = 2 * n * 2.0 ** -53 * (zi.abs().T @ zi.abs())
        assert bool(((kw[i] - ref_w).abs() <= bw).all())
        assert bool(((kz[i] - zi.T @ zi).abs() <= bz).all())
        assert torch.equal(kw[i], kw[i].T) and torch.equal(kz[i], kz[i].T)
