"""The pipelined column passes on grids with an odd nx/2 that no solve on
register tiles takes (in the FP32 form, whose pipeline needs nx/2 even, the
switch changes nothing): bit for bit the plain passes, and the oracle's solve to
the bar of the parity tests (1e-11 in FP64, 1e-5 in FP32).
"""
import numpy as np
import pytest

from oracle import ops
from gpu_util import announce, need_gpu, rel_err, to_np
from test_gpu_fft_pipe import case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,tol", [("FP64", 1e-11), ("FP32_REFINE", 1e-5)])
@pytest.mark.parametrize("shape", [(96, 256, 18), (256, 96, 18), (128, 192, 6)])
def test_pipelined_columns_odd(shape, form, tol):
    torch, m = need_gpu()
    sc = case(shape, 3)
    announce(f"fft pipeline, odd nx/2, {form} {shape}")
    S = m.Solver(sc, precision=getattr(m, form))
    r = np.random.default_rng(22).standard_normal(shape)
    out = []
    for mode in (0, 1):
        S.set_fft_pipeline(mode)
        out.append(to_np(S.poisson(r)))
    S.close()
    assert np.array_equal(out[0], out[1])
    assert rel_err(out[1], ops.poisson_solve(r, sc.spacing)) < tol
