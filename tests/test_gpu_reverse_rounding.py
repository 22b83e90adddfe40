"""The reverse step's rounding: out = fl(fma(c, xprev, fma(a, acc, fl(b x))) + d), acc one FMA an entry in the
row's order, bit for bit against exact rational arithmetic rounded where those operations round.  The
larger product, a acc, is not rounded by itself."""
import ctypes as C
import math
from fractions import Fraction

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _round(v, bits):
    """v to `bits` significant bits, ties to even (no value here is near the ranges' ends)."""
    if v == 0:
        return v
    e = math.frexp(float(v))[1]
    scale = Fraction(2) ** (bits - e)
    return Fraction(round(v * scale)) / scale


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("width", [1, 8, 11])
def test_reverse_step_rounding(precision, width):
    from paper_1504_07690_amd import _abi
    bits, dtype, real = (24, np.float32, C.c_float) if precision == "fp32" else (53, np.float64, C.c_double)
    letter = "f" if precision == "fp32" else "d"
    name = {"f": "_ZN3ssm23launch_reverse_step_f32EliPKiS1_PKffffS3_S3_S3_PfS3_dPdP12ihipStream_tRKNS_8RowOrderE",
            "d": "_ZN3ssm23launch_reverse_step_f64EliPKiS1_PKddddS3_S3_S3_PdS3_dS4_P12ihipStream_tRKNS_8RowOrderE"}
    step = getattr(_abi.lib, name[letter])
    step.restype = C.c_int
    rng = np.random.default_rng(width)
    n, nv = 29, 8
    idx = np.concatenate([np.sort(rng.permutation(n)[:width]) for _ in range(n)]).astype(np.int32)
    ptr = (width * np.arange(n + 1)).astype(np.int32)
    val = rng.standard_normal(n * width).astype(dtype)
    x, xprev, d, y = (rng.standard_normal((n, nv)).astype(dtype) for _ in range(4))
    a, b, c = (dtype(v) for v in (0.37, 0.021, -1.0))
    dev = [torch.tensor(v, device=DEV) for v in (ptr, idx, val, x, xprev, d, np.zeros((n, nv), dtype), y,
                                                 np.zeros(n * width))]
    p = [C.c_void_p(v.data_ptr()) for v in dev]
    order = (C.c_uint64 * 8)()  # the plain order
    err = step(C.c_int64(n), C.c_int(nv), p[0], p[1], p[2], real(a), real(b), real(c), p[3], p[4], p[5], p[6], p[7],
               C.c_double(1.0), p[8], C.c_void_p(torch.cuda.current_stream().cuda_stream), order)
    assert err == 0
    out = dev[6].cpu().numpy()
    F = lambda v: Fraction(float(v))
    want = np.empty_like(out)
    for r in range(n):
        for j in range(nv):
            acc = Fraction(0)
            for e in range(ptr[r], ptr[r + 1]):
                acc = _round(F(val[e]) * F(x[idx[e], j]) + acc, bits)
            t = _round(F(a) * acc + _round(F(b) * F(x[r, j]), bits), bits)
            t = _round(F(c) * F(xprev[r, j]) + t, bits)
            want[r, j] = float(_round(t + F(d[r, j]), bits))
    assert np.array_equal(out, want)
