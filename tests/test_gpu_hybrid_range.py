"""The hybrid term of RESS-DGC at N_v <= 48 where eigenvalues of the pencil are out of range, so that the
in-range eigenvectors of B are wanted, against the oracle.  The degree is too low for the smearing: the
squared filter's first factor is negative in places, where K_W keeps small s_j beside K_Z's entries."""
import numpy as np
import pytest
import torch

from oracle import ssm_oracle as O
from paper_1504_07690_amd import workloads as WL

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("nv,nvh", [(4, 4), (16, 8), (20, 12), (32, 16), (36, 4), (48, 16)])
def test_hybrid_term_with_eigenvalues_out_of_range(nv, nvh):
    from paper_1504_07690_amd import ssm as S
    rng = np.random.default_rng(nv)
    a = WL.laplacian_2d_dirichlet(24, rng.uniform(-1.0, 1.0, size=576))
    lo, hi = WL.interval(a)
    sigma, degree = 0.03 * 0.5 * (hi - lo), 40
    t = 0.5 * (lo + hi) + 0.3 * (hi - lo) * np.linspace(-1.0, 1.0, 9)
    v = WL.gaussian_block(a.n, nv + nvh, seed=nv)
    ref = O.ress_dgc(a, v[:, :nv], v[:, nv:], t, degree, sigma, lo, hi)
    assert nv == 4 or 0 < ref["r2"].sum() < ref["r1"].sum()
    # the inputs decide every test of the ranks by far more than rounding
    g_max = O.range_bound(sigma, a.n)
    bound = 1.001 * g_max
    for i in range(t.size):
        p = O.geneig_trace(ref["k_w"][i], ref["k_z"][i], g_max, return_parts=True, s_floor=ref["floor"][i])[3]
        assert min(np.abs(p["xi"] - bound).min(), np.abs(p["xi"]).min()) > 1e-4 * bound
        assert np.abs(p["s"] - 1e-7 * p["s"].max()).min() > 1e-5 * p["s"].max()
    ctx = S.SSM(S.DeviceCSR.from_csr(a, dtype=torch.float64, device=DEV), lo=lo, hi=hi, sigma=sigma, nv=nv,
                degree=degree, t=t, precision="fp64", w=torch.tensor(v, device=DEV), method="ress", nv_hybrid=nvh,
                device=DEV)
    dos, r1, r2 = ctx.dos()
    assert r1.tolist() == ref["r1"].tolist() and r2.tolist() == ref["r2"].tolist()
    # the bound of the other RESS-DGC tests where the estimate is large
    assert np.abs(dos - ref["dos"]).max() <= 1e-9 * np.abs(ref["dos"]).max()
