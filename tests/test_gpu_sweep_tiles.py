"""The FP32 and FP64 sweep kernel at the edges of its tiles: degree counts around its steps and sets,
point counts around its blocks (dealt evenly to the tiles), column counts around its strips, both
kinds of addressing."""
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _check(precision, kc, ntb, ldc, e, accumulate):
    from paper_1504_07690_amd import ssm as S
    dt = torch.float64 if precision == "fp64" else torch.float32
    g = torch.Generator(device=DEV).manual_seed(kc * 1000 + ntb)
    c = torch.randn(kc, ldc, dtype=dt, device=DEV, generator=g)
    c[:, ntb:] = float("nan")  # the table's padding must not reach a result
    y = torch.randn(kc, e, dtype=dt, device=DEV, generator=g)
    z = torch.randn(ntb, e, dtype=dt, device=DEV, generator=g)
    z0 = z.clone().double()
    S.sweep(precision, c, y, z, accumulate=accumulate)
    eps = torch.finfo(dt).eps
    for q in range(0, e, 1 << 24):  # in pieces: the reference needs 64-bit copies
        yq = y[:, q: q + (1 << 24)].double()
        cq = c[:, :ntb].double()
        base = z0[:, q: q + (1 << 24)] if accumulate else 0.0
        ref = cq.T @ yq + base
        # a sum of kc rounded products in any order, and one more addition
        bound = (kc + 2) * eps * (cq.abs().T @ yq.abs() + (base.abs() if accumulate else 0.0))
        assert bool(((z[:, q: q + (1 << 24)].double() - ref).abs() <= bound).all())


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("kc,ntb,ldc,e", [
    (1, 1, 4, 4), (2, 5, 8, 60), (3, 16, 16, 128), (4, 17, 20, 132), (5, 31, 32, 508), (7, 33, 36, 516),
    (8, 48, 48, 1024), (9, 49, 52, 252), (15, 64, 64, 36), (16, 65, 68, 512), (17, 96, 100, 2052), (31, 97, 100, 260),
    (33, 130, 132, 1028), (64, 205, 208, 388), (65, 8, 8, 40004), (130, 260, 260, 8196)])
def test_sweep_tile_edges(precision, accumulate, kc, ntb, ldc, e):
    _check(precision, kc, ntb, ldc, e, accumulate)


# rows so long that a step's rows span 2^31 bytes: the kernel's 64-bit addresses
@pytest.mark.parametrize("precision,e", [("fp64", (1 << 26) + 2), ("fp32", (1 << 28) + 4)])
def test_sweep_wide_rows(precision, e):
    _check(precision, 3, 2, 4, e, False)


# the same with several tiles of points, added onto Z: every block of points in one tile only
@pytest.mark.parametrize("ntb", [65, 70, 80, 100])
def test_sweep_wide_rows_accumulate(ntb):
    from paper_1504_07690_amd import ssm as S
    kc, e, piece = 3, (1 << 26) + 2, 1 << 23
    g = torch.Generator(device=DEV).manual_seed(ntb)
    c = torch.randn(kc, (ntb + 3) // 4 * 4, dtype=torch.float64, device=DEV, generator=g)
    y = torch.randn(kc, e, dtype=torch.float64, device=DEV, generator=g)

    def start(q):  # of Z's columns q .. q + piece - 1
        col = torch.arange(q, min(q + piece, e), device=DEV, dtype=torch.float64)
        return (1.0 + col % 1024) / 512 - torch.arange(ntb, device=DEV, dtype=torch.float64)[:, None] / 64

    z = torch.empty(ntb, e, dtype=torch.float64, device=DEV)
    for q in range(0, e, piece):
        z[:, q: q + piece] = start(q)
    S.sweep("fp64", c, y, z, accumulate=True)
    cq = c[:, :ntb]
    for q in range(0, e, piece):
        yq, base = y[:, q: q + piece], start(q)
        # a sum of kc rounded products in any order, and one more addition
        bound = (kc + 2) * 2.0 ** -52 * (cq.abs().T @ yq.abs() + base.abs())
        assert bool(((z[:, q: q + piece] - (cq.T @ yq + base)).abs() <= bound).all())
