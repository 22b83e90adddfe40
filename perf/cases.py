"""Workloads of the spectrum sweeping library, timed through its public entry points.

Whole calls (the context's set-up and the DOS; the differentiable DOS forward and
backward) and the stages a program calls on its own buffers: the Chebyshev recurrence,
the sweep, the Gram matrices, Algorithm 4 and the coefficients of Algorithm 1.  The
matrices are the seeded synthetic families of the package (2D Laplacian with a potential,
Anderson lattice, weighted random graph, 27-point lattice), drawn anew for every seed.

listed() names the cases, draw() gives more of the same ranges, prepare() makes a case's
inputs, run() is one pass, work() the bytes and operations it cannot do without, exact()
the same outputs from plain torch and numpy in 64 bits.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1504_07690_amd import workloads as WL

DEV = "cuda:0"
TAU, RHO = 1e-7, 1e-3
ETA_SS = {"fp64": 0.0, "fp32": 2.0 ** -22, "bf16x3": 2.0 ** -16}   # rounding floor, SS-DGC
ETA_RESS = {"fp64": 1e-12, "fp32": 2.0 ** -18}                     # rounding floor, RESS-DGC


def listed():
    return [
        # The paper's small setting, one context's set-up and DOS: latency and launches.
        dict(name="dos_laplace2d_32_fp64", kind="dos", matrix="laplace2d", side=32, nv=40, nvh=0, degree=200, nt=200,
             sigma_hat=0.05, precision="fp64"),
        # The flagship: Anderson lattice, split-BF16 sweep, at a size whose blocks and Z stay resident.
        dict(name="dos_anderson_48_bf16x3", kind="dos", matrix="anderson", side=48, nv=80, nvh=0, degree=1000, nt=500,
             sigma_hat=0.01, precision="bf16x3"),
        # RESS-DGC with the hybrid correction on a random graph: gathers without locality, pair Grams.
        dict(name="dos_graph_ress_fp32", kind="dos", matrix="graph", n=1 << 18, nv=96, nvh=32, degree=300, nt=300,
             sigma_hat=0.02, precision="fp32"),
        # A training step: the differentiable DOS forward and its gradient in every stored value.
        dict(name="grad_anderson_32_fp32", kind="grad", matrix="anderson", side=32, nv=80, degree=300, nt=200,
             sigma_hat=0.02, precision="fp32"),
        # The recurrence alone on the lattice of the benchmark.
        dict(name="chebyshev_anderson_64_fp32", kind="chebyshev", matrix="anderson", side=64, nv=80, degree=64,
             precision="fp32"),
        # The recurrence alone on a random graph, FP64, a ragged row count.
        dict(name="chebyshev_graph_fp64", kind="chebyshev", matrix="graph", n=131101, nv=128, degree=24,
             precision="fp64"),
        # One ring chunk of the split-BF16 sweep at the benchmark's block size.
        dict(name="sweep_bf16x3_large", kind="sweep", n=1 << 18, nv=80, kc=401, ntb=256, degree=1000, sigma_hat=0.01,
             precision="bf16x3"),
        # The FP64 sweep, ragged in every size.
        dict(name="sweep_fp64_ragged", kind="sweep", n=40013, nv=36, kc=333, ntb=205, degree=600, sigma_hat=0.02,
             precision="fp64"),
        # The default precision on a handful of strided sweep points of a large block.
        dict(name="sweep_fp32_few_points", kind="sweep", n=1 << 20, nv=128, kc=32, ntb=8, degree=400, sigma_hat=0.02,
             precision="fp32"),
        # The Gram matrices of a batch of sweep points.
        dict(name="gram_fp32_80", kind="gram", n=1 << 18, nv=80, ntb=125, sigma_hat=0.01, precision="fp32"),
        # Algorithm 4 for a thousand points, some rank deficient.
        dict(name="geneig_128", kind="geneig", nv=128, ntb=1000, sigma_hat=0.005),
        # The coefficient table of the random-graph workload.
        dict(name="coefficients_2000", kind="coefficients", degree=2000, nt=2000, sigma_hat=0.005),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _nv(rng, lo, hi):
    return max(lo, min(hi, 4 * int(round(_log(rng, lo, hi) / 4))))


def draw(rng):
    kind = rng.choice(["dos", "dos", "grad", "chebyshev", "chebyshev", "sweep", "sweep", "gram", "geneig",
                       "coefficients"])
    sigma_hat = round(rng.uniform(0.01, 0.05), 4)
    if kind in ("dos", "grad"):
        matrix = rng.choice(["laplace2d", "anderson", "graph", "stencil27"] if kind == "dos" else
                            ["laplace2d", "anderson"])
        ress = kind == "dos" and rng.random() < 0.4
        c = dict(kind=kind, matrix=matrix)
        if matrix == "laplace2d":
            c["side"] = _log(rng, 24, 160)
        elif matrix == "anderson":
            c["side"] = _log(rng, 10, 40)
        elif matrix == "graph":
            c["n"] = _log(rng, 1000, 100000)
        else:
            c["side"] = rng.choice([16, 18, 24])
        c["nv"] = _nv(rng, 16, 96)
        if kind == "dos":
            c["nvh"] = _nv(rng, 4, 48) if ress else 0
        c["degree"] = 2 * _log(rng, 60, 250)
        c["nt"] = _log(rng, 40, 400)
        c["sigma_hat"] = max(sigma_hat, round(5.0 / c["degree"], 4))
        # RESS-DGC with its FP32 recurrence: in FP64 the moments' rounding is amplified at the spectrum's edges
        c["precision"] = "fp32" if ress else rng.choice(["fp64", "fp32"] + (["bf16x3"] if kind == "dos" else []))
        return c
    if kind == "chebyshev":
        matrix = rng.choice(["laplace2d", "anderson", "graph"])
        c = dict(kind=kind, matrix=matrix)
        if matrix == "laplace2d":
            c["side"] = _log(rng, 24, 400)
        elif matrix == "anderson":
            c["side"] = _log(rng, 10, 60)
        else:
            c["n"] = _log(rng, 1000, 130000)
        c.update(nv=_nv(rng, 8, 128), degree=_log(rng, 8, 48), precision=rng.choice(["fp64", "fp32"]))
        return c
    if kind == "sweep":
        precision = rng.choice(["fp64", "fp32", "bf16x3"])
        degree = _log(rng, 100, 1000)
        return dict(kind=kind, n=_log(rng, 1000, 60000), nv=_nv(rng, 8, 128), kc=min(degree + 1, _log(rng, 24, 400)),
                    ntb=_log(rng, 5, 300), degree=degree, sigma_hat=sigma_hat, precision=precision)
    if kind == "gram":
        return dict(kind=kind, n=_log(rng, 1000, 200000), nv=_nv(rng, 16, 256), ntb=_log(rng, 4, 64),
                    sigma_hat=sigma_hat, precision=rng.choice(["fp64", "fp32"]))
    if kind == "geneig":
        nv = _nv(rng, 16, 200)
        return dict(kind=kind, nv=nv, ntb=_log(rng, 16, 1000 if nv <= 128 else 250), sigma_hat=sigma_hat)
    return dict(kind=kind, degree=_log(rng, 50, 2000), nt=_log(rng, 20, 2000), sigma_hat=sigma_hat)


# ----------------------------------------------------------------------------
# Inputs
# ----------------------------------------------------------------------------
def _dtype(precision):
    return torch.float64 if precision == "fp64" else torch.float32


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _matrix(case, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    kind = case["matrix"]
    if kind == "laplace2d":
        side = case["side"]
        return WL.laplacian_2d_dirichlet(side, rng.uniform(-1.0, 1.0, size=side * side)), None
    if kind == "anderson":
        side = case["side"]
        return WL.anderson_3d(side, rng.uniform(-2.0, 2.0, size=side ** 3)), (side, side, side)
    if kind == "graph":
        return WL.er_graph_laplacian(case["n"], 16, rng), None
    side = case["side"]
    return WL.stencil27_lognormal(side, rng), (side, side, side)


def _points(case, lo, hi, nt):
    """Sweep points: the midpoints of [lo, hi]; for a gradient those of its middle half, inside the spectrum."""
    grid = -1.0 + (2.0 * np.arange(nt) + 1.0) / nt
    return 0.5 * (lo + hi) + 0.5 * (hi - lo) * (0.5 if case["kind"] == "grad" else 1.0) * grid


def _table(t, degree, sigma, n, lo, hi):
    """Coefficients of Algorithm 1, (degree + 1) x nt in FP64, by the DFT of its definition."""
    two = 1
    while two < 4 * (degree + 1):
        two *= 2
    theta = torch.arange(two, dtype=torch.float64, device=DEV) * (2.0 * math.pi / two)
    x = 0.5 * (lo + hi) + 0.5 * (hi - lo) * torch.cos(theta)
    t = torch.as_tensor(np.asarray(t), dtype=torch.float64, device=DEV)
    g = torch.exp(-(t[:, None] - x[None, :]) ** 2 / (2.0 * sigma * sigma)) / (n * math.sqrt(2.0 * math.pi) * sigma)
    mu = torch.fft.fft(g, dim=1).real[:, : degree + 1] / two
    mu[:, 1:] *= 2.0
    return mu.T.contiguous()


def _sweep_inputs(case, seed):
    """A coefficient table (kc x ldc) and a chunk of blocks with entries of the size of T_k(A~)W's."""
    nt, e = case["ntb"], case["n"] * case["nv"]
    t = -1.0 + (2.0 * np.arange(nt) + 1.0) / nt
    c = torch.zeros(case["kc"], (nt + 3) // 4 * 4, dtype=torch.float64, device=DEV)
    c[:, :nt] = _table(t, case["degree"], case["sigma_hat"], case["n"], -1.0, 1.0)[: case["kc"]]
    y = torch.randn(case["kc"], e, dtype=_dtype(case["precision"]), device=DEV, generator=_generator(seed))
    return c, y


def _gram_inputs(case, seed):
    """W and Z_i = g(t_i I - D) W for a diagonal operator D: W^T Z_i is symmetric as on the method's path."""
    g = _generator(seed)
    n, nv, nt = case["n"], case["nv"], case["ntb"]
    dt = _dtype(case["precision"])
    w = torch.randn(n, nv, dtype=dt, device=DEV, generator=g)
    lam = 1.8 * torch.rand(n, dtype=torch.float64, device=DEV, generator=g) - 0.9
    z = torch.empty(nt, n, nv, dtype=dt, device=DEV)
    for i in range(nt):
        t = -0.9 + 1.8 * (i + 0.5) / nt
        z[i] = w * (torch.exp(-(t - lam) ** 2 / (2.0 * case["sigma_hat"] ** 2)) / n).to(dt)[:, None]
    return w, z


def _pencils(case, seed):
    """K_W = W^T g W and K_Z = W^T g^2 W of a diagonal operator with 4096 random eigenvalues, and max g."""
    g = _generator(seed)
    n, nv, nt, s = 4096, case["nv"], case["ntb"], case["sigma_hat"]
    w = torch.randn(n, nv, dtype=torch.float64, device=DEV, generator=g)
    lam = 1.8 * torch.rand(n, dtype=torch.float64, device=DEV, generator=g) - 0.9
    g_max = 1.0 / (n * math.sqrt(2.0 * math.pi) * s)
    kw = torch.empty(nt, nv, nv, dtype=torch.float64, device=DEV)
    kz = torch.empty_like(kw)
    for i in range(nt):
        t = -0.9 + 1.8 * (i + 0.5) / nt
        zi = w * (g_max * torch.exp(-(t - lam) ** 2 / (2.0 * s * s)))[:, None]
        kw[i] = w.T @ zi
        kz[i] = zi.T @ zi
    return 0.5 * (kw + kw.mT), 0.5 * (kz + kz.mT), g_max


def _problem(case, seed):
    """Matrix, interval, smearing, sweep points and random block of a whole call."""
    a, lattice = _matrix(case, seed)
    lo, hi = WL.interval(a)
    w = torch.randn(a.n, case["nv"] + case.get("nvh", 0), dtype=_dtype(case["precision"]), device=DEV,
                    generator=_generator(seed))
    return a, lattice, lo, hi, case["sigma_hat"] * 0.5 * (hi - lo), _points(case, lo, hi, case["nt"]), w


def prepare(case, seed):
    from paper_1504_07690_amd import ssm as S
    kind = case["kind"]
    if kind == "dos":
        a, lattice, lo, hi, sigma, t, w = _problem(case, seed)
        csr = S.DeviceCSR.from_csr(a, dtype=_dtype(case["precision"]))
        ctx = S.SSM(csr, lo=lo, hi=hi, sigma=sigma, nv=case["nv"], degree=case["degree"], t=t,
                    precision=case["precision"], w=w, method="ress" if case["nvh"] else "ss", nv_hybrid=case["nvh"],
                    lattice=lattice)
        return dict(case=case, S=S, ctx=ctx)
    if kind == "grad":
        a, lattice, lo, hi, sigma, t, w = _problem(case, seed)
        csr = S.DeviceCSR.from_csr(a, dtype=_dtype(case["precision"]))
        values = csr.values.clone().requires_grad_(True)
        # the weights of a smooth function of the spectrum
        weight = torch.as_tensor(np.cos(np.linspace(0.0, 3.0, case["nt"])), device=DEV)
        opts = dict(lo=lo, hi=hi, sigma=sigma, nv=case["nv"], degree=case["degree"], t=t,
                    precision=case["precision"], w=w, lattice=lattice)
        return dict(case=case, S=S, csr=csr, values=values, weight=weight, opts=opts)
    if kind == "chebyshev":
        a, _ = _matrix(case, seed)
        lo, hi = WL.interval(a)
        dt = _dtype(case["precision"])
        w = torch.randn(a.n, case["nv"], dtype=dt, device=DEV, generator=_generator(seed))
        y = torch.empty(case["degree"] + 1, a.n, case["nv"], dtype=dt, device=DEV)
        return dict(case=case, S=S, csr=S.DeviceCSR.from_csr(a, dtype=dt), lo=lo, hi=hi, w=w, y=y)
    if kind == "sweep":
        c, y = _sweep_inputs(case, seed)
        st = dict(case=case, S=S, y=y, z=torch.empty(case["ntb"], y.shape[1], dtype=y.dtype, device=DEV))
        if case["precision"] == "bf16x3":
            kmax = c.abs().amax(dim=1)
            st["k3"] = int(torch.nonzero(kmax >= kmax.max() * 2.0 ** -8).max()) + 1
            st["chi"], st["clo"] = S.split_coefficients(c, case["ntb"], (case["kc"] + 63) // 64 * 64)
        else:
            st["c"] = c.to(y.dtype)
        return st
    if kind == "gram":
        w, z = _gram_inputs(case, seed)
        nn = (case["ntb"], case["nv"], case["nv"])
        segs = min(64, max(1, (1024 + case["ntb"] - 1) // case["ntb"]))
        while segs > 1 and case["n"] // segs < 256:
            segs -= 1
        return dict(case=case, S=S, w=w, z=z, segs=segs, kw=torch.empty(nn, dtype=torch.float64, device=DEV),
                    kz=torch.empty(nn, dtype=torch.float64, device=DEV))
    if kind == "geneig":
        kw, kz, g_max = _pencils(case, seed)
        return dict(case=case, S=S, kw=kw, kz=kz, g_max=g_max,
                    dos=torch.empty(case["ntb"], dtype=torch.float64, device=DEV),
                    ranks=torch.empty(2 * case["ntb"], dtype=torch.int32, device=DEV))
    t = _coefficient_points(case, seed)
    return dict(case=case, S=S, t=torch.as_tensor(t, device=DEV),
                c=torch.empty(case["degree"] + 1, case["nt"], dtype=torch.float64, device=DEV),
                c32=torch.empty(case["degree"] + 1, case["nt"], dtype=torch.float32, device=DEV))


def _coefficient_points(case, seed):
    return np.sort(np.random.Generator(np.random.PCG64(seed)).uniform(-1.0, 1.0, case["nt"]))


# ----------------------------------------------------------------------------
# One pass
# ----------------------------------------------------------------------------
def run(state):
    case, S = state["case"], state["S"]
    kind = case["kind"]
    if kind == "dos":
        state["ctx"].reset()
        dos, r1, r2 = state["ctx"].dos()
        return {"dos": dos, "r1": r1, "r2": r2}
    if kind == "grad":
        csr = state["csr"]
        dos = S.dos_autograd(state["values"], csr.row_ptr, csr.col_idx, csr.n, **state["opts"])
        (grad,) = torch.autograd.grad(dos, state["values"], state["weight"])
        return {"dos": dos.detach(), "grad": grad}
    if kind == "chebyshev":
        S.chebyshev(state["csr"], state["lo"], state["hi"], case["precision"], state["w"], state["y"])
        return {"y": state["y"]}
    if kind == "sweep":
        if case["precision"] == "bf16x3":
            S.sweep_split(state["chi"], state["clo"], state["y"], state["z"], k3=state["k3"])
        else:
            S.sweep(case["precision"], state["c"], state["y"], state["z"])
        return {"z": state["z"]}
    if kind == "gram":
        S.gram(case["precision"], state["w"], state["z"], state["kw"], state["kz"], nseg=state["segs"])
        return {"k_w": state["kw"], "k_z": state["kz"]}
    if kind == "geneig":
        S.geneig_trace(state["kw"], state["kz"], state["g_max"], TAU, RHO, state["dos"], state["ranks"])
        return {"dos": state["dos"], "ranks": state["ranks"]}
    S.coefficients(-1.0, 1.0, case["sigma_hat"], 4096, state["t"], case["degree"], state["c"], state["c32"])
    return {"c": state["c"], "c32": state["c32"]}


# ----------------------------------------------------------------------------
# What a pass cannot do without
# ----------------------------------------------------------------------------
def _size(case):
    """Rows and (about) stored entries of a case's matrix."""
    kind = case["matrix"]
    n = case["n"] if kind == "graph" else case["side"] ** (2 if kind == "laplace2d" else 3)
    return n, n * {"laplace2d": 5, "anderson": 7, "graph": 17, "stencil27": 27}[kind]


def work(case):
    kind = case["kind"]
    es = 8 if case.get("precision") == "fp64" else 4
    if kind in ("dos", "grad"):
        n, nnz = _size(case)
        nv, nt, m = case["nv"] + case.get("nvh", 0), case["nt"], case["degree"]
        if case.get("nvh"):
            h = m // 2 + 1
            flops = 2.0 * nnz * nv * h + 2.0 * n * nv * nv * h + 2.0 * nt * nv * nv * (m + h)
        else:
            flops = 2.0 * nnz * nv * m + 2.0 * n * nv * (m + 1) * nt + 2.0 * n * nv * nv * nt
        flops += 12.0 * nt * case["nv"] ** 3
        nbytes = nnz * (4 + es) + n * nv * es + nt * 24
        if kind == "grad":
            flops += 4.0 * nnz * nv * m + 2.0 * n * nv * (m + 1) * nt + 4.0 * n * nv * nv * nt
            nbytes += nnz * es
        return {"bytes": nbytes, "flops": flops}
    if kind == "chebyshev":
        n, nnz = _size(case)
        return {"bytes": nnz * (4 + es) + n * case["nv"] * es * (case["degree"] + 2),
                "flops": 2.0 * nnz * case["nv"] * case["degree"]}
    if kind == "sweep":
        e = case["n"] * case["nv"]
        return {"bytes": (case["kc"] + case["ntb"]) * e * es + case["kc"] * case["ntb"] * es,
                "flops": 2.0 * e * case["kc"] * case["ntb"]}
    if kind == "gram":
        n, nv = case["n"], case["nv"]
        return {"bytes": (case["ntb"] + 1) * n * nv * es + case["ntb"] * 2 * nv * nv * 8,
                "flops": 2.0 * n * nv * nv * case["ntb"]}
    if kind == "geneig":
        nv = case["nv"]
        return {"bytes": case["ntb"] * 2 * nv * nv * 8, "flops": 12.0 * case["ntb"] * nv ** 3}
    m1, nt = case["degree"] + 1, case["nt"]
    return {"bytes": nt * 8 + m1 * nt * 12, "flops": nt * (20.0 * m1 + 10.0 * m1 * math.log2(4 * m1))}


# ----------------------------------------------------------------------------
# The same outputs in 64 bits
# ----------------------------------------------------------------------------
def _csr64(a, precision):
    """The stored values as the pass sees them (rounded to FP32 outside fp64), in 64 bits."""
    vals = a.values if precision == "fp64" else a.values.astype(np.float32).astype(np.float64)
    return torch.sparse_csr_tensor(torch.as_tensor(a.row_ptr.astype(np.int64)),
                                   torch.as_tensor(a.col_idx.astype(np.int64)), torch.as_tensor(vals),
                                   size=(a.n, a.n)).to(DEV)


def _blocks(a64, w64, lo, hi, degree):
    """T_k(A~) W for k = 0..degree."""
    alpha, beta = 2.0 / (hi - lo), -(hi + lo) / (hi - lo)
    prev, cur = None, w64
    yield cur
    for k in range(degree):
        nxt = alpha * (a64 @ cur) + beta * cur
        prev, cur = cur, (nxt if k == 0 else 2.0 * nxt - prev)
        yield cur


def _filtered(a64, w64, lo, hi, c):
    """Z_i = sum_k c[k, i] T_k(A~) W, the blocks taken a few at a time, and W^T T_k(A~) W of each k."""
    m1, nt = c.shape
    z = torch.zeros(nt, w64.numel(), dtype=torch.float64, device=DEV)
    step = max(1, min(64, int(4e9 / (8 * w64.numel()))))
    moments, held, k0 = [], [], 0
    for k, y in enumerate(_blocks(a64, w64, lo, hi, m1 - 1)):
        moments.append(w64.T @ y)
        held.append(y.reshape(-1))
        if len(held) == step or k == m1 - 1:
            z.addmm_(c[k0: k + 1].T, torch.stack(held))
            held, k0 = [], k + 1
    return z, moments


def _pencil_trace(kw, kz, g_max, s_floor=0.0):
    """Algorithm 4 for one point: the trace and C~ = U~ S~^-1/2 Q~ of the kept pairs."""
    s, u = np.linalg.eigh(0.5 * (kw + kw.T))
    if not s.max() > 0.0:
        return 0.0, np.zeros((len(s), 0))
    keep = (s >= TAU * s.max()) & (s >= s_floor)
    if not keep.any():
        return 0.0, np.zeros((len(s), 0))
    ut = u[:, keep] / np.sqrt(s[keep])
    b = ut.T @ kz @ ut
    xi, q = np.linalg.eigh(0.5 * (b + b.T))
    ok = (xi >= 0.0) & (xi <= (1.0 + RHO) * g_max)
    return float(xi[ok].sum()), ut @ q[:, ok]


def _exact_dos(case, seed):
    a, _, lo, hi, sigma, t, w = _problem(case, seed)
    n, nv, nvh, m = a.n, case["nv"], case["nvh"], case["degree"]
    a64, w64 = _csr64(a, case["precision"]), w.double()
    c = _table(t, m, sigma, n, lo, hi)
    if nvh:
        c = c[: m // 2 + 1]
    z, x = _filtered(a64, w64, lo, hi, c)
    z = z.view(case["nt"], n, nv + nvh)
    if nvh:
        xmax = torch.stack([v[:nv, :nv].abs().max() for v in x])
        floor = (ETA_RESS[case["precision"]] * (c.abs() * xmax[:, None]).sum(dim=0)).cpu().numpy()
    else:
        floor = (ETA_SS[case["precision"]] * c.square().sum(dim=0).sqrt() * w64.square().sum()
                 / math.sqrt(n * nv)).cpu().numpy()
    g_max = 1.0 / (n * math.sqrt(2.0 * math.pi) * sigma)
    dos = np.zeros(case["nt"])
    for i in range(case["nt"]):
        kvv = (w64.T @ z[i]).cpu().numpy()
        zw = z[i, :, :nv]
        kz = (zw.T @ zw).cpu().numpy()
        dos[i], cc = _pencil_trace(kvv[:nv, :nv], kz, g_max, floor[i])
        if nvh:
            kc = kvv[nv:, :nv] @ cc
            dos[i] += (np.trace(kvv[nv:, nv:]) - np.sum(kc * kc)) / nvh
    return {"dos": dos, "r1": None, "r2": None}


def _exact_grad(case, seed):
    """The DOS, and the gradient of sum_i weight_i dos_i with the kept sets of Algorithm 4 frozen."""
    a, _, lo, hi, sigma, t, w = _problem(case, seed)
    n, nv, m, nt = a.n, case["nv"], case["degree"], case["nt"]
    a64, w64 = _csr64(a, case["precision"]), w.double()
    c = _table(t, m, sigma, n, lo, hi)
    z, _ = _filtered(a64, w64, lo, hi, c)
    z = z.view(nt, n, nv)
    floor = (ETA_SS[case["precision"]] * c.square().sum(dim=0).sqrt() * w64.square().sum()
             / math.sqrt(n * nv)).cpu().numpy()
    g_max = 1.0 / (n * math.sqrt(2.0 * math.pi) * sigma)
    weight = np.cos(np.linspace(0.0, 3.0, nt))
    dos = np.zeros(nt)
    for i in range(nt):
        kw = (w64.T @ z[i]).cpu().numpy()
        kz = (z[i].T @ z[i]).cpu().numpy()
        s, u = np.linalg.eigh(0.5 * (kw + kw.T))
        keep = (s >= TAU * s.max()) & (s >= floor[i]) & (s.max() > 0.0)
        f = np.where(keep, 1.0 / np.sqrt(np.where(keep, s, 1.0)), 0.0)
        kt = u.T @ kz @ u
        b = (f[:, None] * kt * f[None, :])[np.ix_(keep, keep)]
        xi, q = np.linalg.eigh(0.5 * (b + b.T))
        ok = (xi >= 0.0) & (xi <= (1.0 + RHO) * g_max)
        dos[i] = xi[ok].sum()
        p = np.zeros((nv, nv))
        p[np.ix_(keep, keep)] = q[:, ok] @ q[:, ok].T
        r = np.sqrt(np.where(keep, s, 1.0))
        with np.errstate(divide="ignore", invalid="ignore"):
            mixed = (f[:, None] - f[None, :]) / (s[:, None] - s[None, :])
        both = keep[:, None] & keep[None, :]
        gamma = np.where(both, -1.0 / (np.outer(r, r) * (r[:, None] + r[None, :])),
                         np.where(keep[:, None] | keep[None, :], mixed, 0.0))
        kdp = kt @ (f[:, None] * p)
        kwb = weight[i] * u @ (gamma * (kdp + kdp.T)) @ u.T
        kzb = weight[i] * u @ (f[:, None] * p * f[None, :]) @ u.T
        z[i] = w64 @ torch.as_tensor(kwb, device=DEV) + 2.0 * (z[i] @ torch.as_tensor(kzb, device=DEV))
    alpha, beta = 2.0 / (hi - lo), -(hi + lo) / (hi - lo)
    ys = list(_blocks(a64, w64, lo, hi, m))
    rows = torch.as_tensor(np.repeat(np.arange(n), np.diff(a.row_ptr)), device=DEV)
    cols = torch.as_tensor(a.col_idx.astype(np.int64), device=DEV)
    grad = torch.zeros(a.nnz, dtype=torch.float64, device=DEV)
    zero = torch.zeros_like(w64)
    l1, l2 = zero, zero
    flat = z.view(nt, -1)
    for k in range(m, 0, -1):
        lam = (c[k][None, :] @ flat).view(n, nv) + 2.0 * (alpha * (a64 @ l1) + beta * l1) - l2
        y = ys[k - 1]
        for e0 in range(0, a.nnz, 1 << 21):
            sl = slice(e0, e0 + (1 << 21))
            grad[sl] += (1.0 if k == 1 else 2.0) * alpha * (lam[rows[sl]] * y[cols[sl]]).sum(dim=1)
        l1, l2 = lam, l1
    return {"dos": torch.as_tensor(dos), "grad": grad}


def exact(case, seed):
    kind = case["kind"]
    if kind == "dos":
        return _exact_dos(case, seed)
    if kind == "grad":
        return _exact_grad(case, seed)
    if kind == "chebyshev":
        a, _ = _matrix(case, seed)
        lo, hi = WL.interval(a)
        w = torch.randn(a.n, case["nv"], dtype=_dtype(case["precision"]), device=DEV, generator=_generator(seed))
        y = torch.empty(case["degree"] + 1, a.n, case["nv"], dtype=torch.float64, device=DEV)
        for k, b in enumerate(_blocks(_csr64(a, case["precision"]), w.double(), lo, hi, case["degree"])):
            y[k] = b
        return {"y": y}
    if kind == "sweep":
        c, y = _sweep_inputs(case, seed)
        # the split tables are made from the FP64 coefficients, the others rounded to the blocks' type
        c64 = (c if case["precision"] == "bf16x3" else c.to(y.dtype).double())[:, : case["ntb"]].T.contiguous()
        z = torch.empty(case["ntb"], y.shape[1], dtype=torch.float64, device=DEV)
        for q in range(0, y.shape[1], 1 << 20):
            z[:, q: q + (1 << 20)] = c64 @ y[:, q: q + (1 << 20)].double()
        return {"z": z}
    if kind == "gram":
        w, z = _gram_inputs(case, seed)
        nv = case["nv"]
        blk = torch.arange(nv, device=DEV) // 16
        upper, same = blk[:, None] < blk[None, :], blk[:, None] == blk[None, :]
        kw, kz = [], []
        for i in range(case["ntb"]):
            zi = z[i].double()
            m = w.double().T @ zi
            # the stated completion: upper 16 x 16 blocks, mirrored, the diagonal ones averaged
            kw.append(torch.where(upper, m, torch.where(same, 0.5 * (m + m.T), m.T)))
            kz.append(zi.T @ zi)
        return {"k_w": torch.stack(kw), "k_z": torch.stack(kz)}
    if kind == "geneig":
        if case["ntb"] * case["nv"] ** 3 > 2.5e9:
            return None
        kw, kz, g_max = (v.cpu().numpy() if torch.is_tensor(v) else v for v in _pencils(case, seed))
        return {"dos": torch.as_tensor([_pencil_trace(kw[i], kz[i], g_max)[0] for i in range(case["ntb"])],
                                       dtype=torch.float64), "ranks": None}
    c = _table(_coefficient_points(case, seed), case["degree"], case["sigma_hat"], 4096, -1.0, 1.0)
    return {"c": c, "c32": c}
