"""The coefficient kernel's transform at the edges of its sizes: every radix that ends it (2N_theta
is the least power of two >= 4 (M + 1)), one point and point counts around the split over XCDs."""
import numpy as np
import pytest
import torch

from oracle import ssm_oracle as O
from paper_1504_07690_amd import workloads as WL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("degree,nt", [(1, 1), (2, 9), (3, 8), (4, 7), (7, 64), (8, 65), (15, 3), (31, 17), (63, 2),
                                       (64, 511), (127, 5), (255, 12), (511, 4), (512, 1030), (1023, 6), (1024, 10),
                                       (2047, 515), (2048, 259), (4095, 9)])
def test_coefficients_every_transform_size(degree, nt):
    from paper_1504_07690_amd import ssm as S
    lo, hi, n, sigma = -1.0, 1.0, 4096, 0.05
    t = WL.midpoint_grid(nt)
    c = torch.full((degree + 1, nt), 7.0, dtype=torch.float64, device="cuda:0")
    c32 = torch.full((degree + 1, nt), 7.0, dtype=torch.float32, device="cuda:0")
    S.coefficients(lo, hi, sigma, n, torch.tensor(t, device="cuda:0"), degree, c, c32)
    ref = O.dgc_coefficients(t, degree, sigma, n, lo, hi)
    # g's own rounding, about 0.6 |t| / sigma eps, and a few eps per pass of each side's transform
    assert np.abs(c.cpu().numpy() - ref).max() <= 1e-13 * O.range_bound(sigma, n)
    assert np.array_equal(c32.cpu().numpy(), c.cpu().numpy().astype(np.float32))
