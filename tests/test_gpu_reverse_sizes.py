"""The reverse recurrence at the edges of its row groups: one to sixteen rows a wave, rows of no, few,
eight, nine and many entries, ragged row counts, against central differences of the estimate itself.
The Gaussians are wide and N_v is small beside the eigenvalues under them, so no eigenvalue is cut off
and the estimate is smooth."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
M, NT = 30, 3


def _matrix(n, rng):
    """Symmetric pattern: a ring, row 0 without entries but its diagonal's absence, one row of 9 and
    one of 30 entries."""
    ent = {}
    for i in range(1, n):
        for j in ((i + 1) % n, (i + 2) % n, i):
            if j == 0 or i == 0:
                continue
            ent[i, j] = ent[j, i] = rng.uniform(-0.4, 0.4)
    for row, want in ((n // 2, 9), (n // 3, 30)):
        have = [j for (i, j) in ent if i == row]
        for j in rng.permutation(np.arange(1, n)):
            if len(have) >= min(want, n - 1):
                break
            if (row, int(j)) not in ent:
                ent[row, int(j)] = ent[int(j), row] = rng.uniform(-0.2, 0.2)
                have.append(j)
    keys = sorted(ent)
    ptr = np.searchsorted([k[0] for k in keys], np.arange(n + 1))
    return ptr, np.array([k[1] for k in keys]), np.array([ent[k] for k in keys]), {k: e for e, k in enumerate(keys)}


def _run(S, n, ptr, idx, val, nv, precision, w, weight, grad, lattice=None):
    dtype = torch.float64 if precision == "fp64" else torch.float32
    csr = S.DeviceCSR(n, ptr, idx, val, dtype=dtype)
    ctx = S.SSM(csr, lo=-4.0, hi=4.0, sigma=1.2, nv=nv, degree=M, t=np.array([-1.0, 0.1, 1.2]), precision=precision,
                w=w.to(dtype), lattice=lattice)
    dos, r1, _ = ctx.dos()
    assert (r1 == nv).all()
    f = float(np.dot(weight, dos))
    return (f, ctx.backward(weight).cpu().numpy()) if grad else f


@pytest.mark.parametrize("nv", [4, 12, 16, 20, 40, 44, 80, 88, 132, 256])
def test_reverse_sizes(nv):
    from paper_1504_07690_amd import ssm as S
    rng = np.random.default_rng(nv)
    n = 12 * nv + 37
    ptr, idx, val, where = _matrix(n, rng)
    w = torch.tensor(rng.standard_normal((n, nv)), device=DEV)
    weight = np.array([1.0, -0.7, 0.4])
    f, g = _run(S, n, ptr, idx, val, nv, "fp64", w, weight, True)
    _, g32 = _run(S, n, ptr, idx, val, nv, "fp32", w, weight, True)
    assert np.linalg.norm(g32 - g) <= 1e-3 * np.linalg.norm(g)
    long_row, nine = n // 3, n // 2
    picks = [np.isin(np.arange(len(val)), np.arange(ptr[r], ptr[r + 1])[sl])
             for r, sl in ((long_row, slice(0, 8)), (long_row, slice(8, 16)), (long_row, slice(16, None)),
                           (nine, slice(8, None)), (nine, slice(0, 8)))] + [np.ones(len(val), bool)]
    rows = np.repeat(np.arange(n), np.diff(ptr))
    for pick in picks:
        d = rng.standard_normal(len(val)) * pick
        for e in np.flatnonzero(pick):  # the estimate is defined on symmetric matrices
            d[where[int(idx[e]), int(rows[e])]] = d[e]
        h = 1e-3 / np.linalg.norm(d)
        diff = []
        for s in (h, 2 * h):
            hi, lo = (_run(S, n, ptr, idx, val + sg * s * d, nv, "fp64", w, weight, False) for sg in (1, -1))
            diff.append((hi - lo) / (2 * s))
        # the difference's own error: a third of what halving the step changed, and rounding of f
        tol = 2 * abs(diff[0] - diff[1]) + 1e4 * 2.0 ** -52 * abs(f) / h
        assert abs(float(np.dot(g, d)) - diff[0]) <= tol


@pytest.mark.parametrize("nv", [16, 40, 80])
def test_reverse_order_of_rows(nv):
    """A lattice's tiled order gives the same bits as plain order."""
    from paper_1504_07690_amd import ssm as S, workloads as WL
    rng = np.random.default_rng(1)
    a = WL.anderson_3d(12, rng.uniform(-2.0, 2.0, size=12 ** 3))
    w = torch.tensor(rng.standard_normal((a.n, nv)), device=DEV)
    weight = np.ones(NT)
    out = []
    for lattice in (None, (12, 12, 12)):
        csr = S.DeviceCSR.from_csr(a, dtype=torch.float64)
        lo, hi = WL.interval(a)
        ctx = S.SSM(csr, lo=lo, hi=hi, sigma=0.15 * (hi - lo), nv=nv, degree=M, t=np.linspace(-2.0, 2.0, NT),
                    precision="fp64", w=w, lattice=lattice)
        ctx.dos()
        out.append(ctx.backward(weight))
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("part", [False, True])
@pytest.mark.parametrize("nv", [56, 128, 136])
def test_backward_with_eigenvalues_out_of_range(nv, part):
    """Algorithm 4's backward above N_v = 48 against the Jacobi kernel's: W's 44 columns padded with zero
    columns, whose eigenvalues are cut off, give the same gradient.  Once with every eigenvalue of the
    pencil in range, once with K_Z scaled so that the range's upper end is in their widest gap."""
    from paper_1504_07690_amd import ssm as S
    rng = np.random.default_rng(nv)
    n, base = 400, 44
    ptr, idx, val, _ = _matrix(n, rng)
    w = torch.tensor(rng.standard_normal((n, base)), device=DEV)
    weight = np.array([1.0, -0.7, 0.4])
    grads, conds, scale = [], [], None
    for cols in (base, nv):
        ctx = S.SSM(S.DeviceCSR(n, ptr, idx, val, dtype=torch.float64), lo=-4.0, hi=4.0, sigma=1.2, nv=cols, degree=M,
                    t=np.array([-1.0, 0.1, 1.2]), precision="fp64",
                    w=torch.cat([w, torch.zeros(n, cols - base, dtype=w.dtype, device=DEV)], 1).contiguous())
        _, r1, r2 = ctx.dos()
        assert (r1 == base).all() and (r2 == base).all()
        v = ctx.views()
        if scale is None:
            kw, kz = v["k_w"].cpu().numpy(), v["k_z"].cpu().numpy()
            s, u = np.linalg.eigh(0.5 * (kw + kw.transpose(0, 2, 1)))
            conds = s[:, -1] / s[:, 0]
            half = u / np.sqrt(s)[:, None, :]
            xi = np.linalg.eigvalsh(half.transpose(0, 2, 1) @ kz @ half)
            mid = xi[:, base // 4: 3 * base // 4]
            gap = np.diff(mid, axis=1).argmax(1)
            end = 0.5 * (mid[np.arange(NT), gap] + mid[np.arange(NT), gap + 1])
            g_max = 1.0 / (n * np.sqrt(2 * np.pi) * 1.2)
            scale = torch.tensor(1.001 * g_max / end if part else np.ones(NT), device=DEV)
        v["k_z"].mul_(scale[:, None, None])
        grads.append(ctx.backward(weight).cpu().numpy())
    # rounding of K_W over its smallest eigenvalue, to the power in F's differences; scaled K_Z
    tol = 500 * 2.0 ** -52 * conds.max() ** 1.5 * max(1.0, float(scale.max()))
    assert np.linalg.norm(grads[1] - grads[0]) <= tol * np.linalg.norm(grads[0])
