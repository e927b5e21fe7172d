"""The filter and the correction at the sizes where their launch changes: the
small tiles with chunks of 2 and 4 planes, the register-ring forms from 2^20
cells on with a shorter last chunk and with a single chunk, and grids that the
64 x 16 tile does not divide.

Tolerances: those of the operator tests, 1e-13 (FP64) and 1e-5 (FP32 form) of
the largest value.
"""
import numpy as np
import pytest

from oracle import ops
from gpu_util import announce, need_gpu, rel_err, to_np
from test_gpu_parity import make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,tol", [("FP64", 1e-13), ("FP32_REFINE", 1e-5)])
@pytest.mark.parametrize("shape", [(3, 64, 64), (64, 64, 128), (54, 48, 192), (162, 128, 64), (4, 512, 512),
                                   (72, 108, 162), (1, 192, 256)])
def test_filter(shape, form, tol):
    torch, m = need_gpu()
    sc = make_case(shape, 9)
    announce(f"filter chunks {shape} {form}")
    S = m.Solver(sc, precision=getattr(m, form))
    assert rel_err(to_np(S.filter(sc.c)), sc.beta * ops.filter6(sc.c, sc.spacing)) < tol
    S.close()
