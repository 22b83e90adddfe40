"""Algorithm 4 at N_v <= 48 where the one-workgroup kernel hands a point to the Jacobi kernel: zero, not
finite, and far out of scale, next to ordinary points."""
import numpy as np
import pytest
import torch

from oracle import ssm_oracle as O

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("nv", [1, 2, 16, 17, 33, 48])
def test_geneig_points_left_to_jacobi(nv):
    from paper_1504_07690_amd import ssm as S
    rng = np.random.default_rng(100 + nv)
    w = rng.standard_normal((300, nv))
    z = w * rng.uniform(0.05, 0.95, 300)[:, None]
    k_w, k_z = w.T @ z, z.T @ z
    kw, kz = np.stack([k_w] * 8), np.stack([k_z] * 8)
    kw[1], kz[1] = 0.0, 0.0
    kw[2] *= 2.0 ** -400
    kz[2] *= 2.0 ** -400
    kw[3] *= 2.0 ** 400
    kz[3] *= 2.0 ** 400
    kw[4][0, 0] = np.nan
    kz[5][nv - 1, 0] = kz[5][0, nv - 1] = np.inf
    kz[6] = 0.0
    dos = torch.full((8,), 7.0, dtype=torch.float64, device=DEV)
    ranks = torch.full((16,), -1, dtype=torch.int32, device=DEV)
    S.geneig_trace(torch.tensor(kw, device=DEV), torch.tensor(kz, device=DEV), 1.0, 1e-7, 1e-3, dos, ranks)
    out = dos.cpu().numpy()
    ok = [0, 1, 2, 3, 6, 7]
    ref = [O.geneig_trace(kw[i], kz[i], 1.0) for i in ok]
    # full rank, well conditioned K_W: 500 units of rounding in each of nv eigenvalues <= 1
    assert np.abs(out[ok] - [r[0] for r in ref]).max() <= 500 * 2.0 ** -52 * nv * np.linalg.cond(k_w)
    assert ranks[ok[:4]].tolist() == [r[1] for r in ref[:4]]
    assert ranks[8:].cpu().numpy()[ok[:4]].tolist() == [r[2] for r in ref[:4]]
