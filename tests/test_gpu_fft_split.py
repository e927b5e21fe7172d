"""The three-pass FFT solve (the y transform split between the x passes and the
z pass) against the oracle's Poisson solve (Section 2.2).

The shapes (nz, ny, nx) take every compiled x length nx/2, every factor pair
(R, Q) of ny and every z length once or more, with cells of unequal sides, in
both precisions; the bar is that of the FFT solve's parity tests (1e-11 in FP64,
1e-5 in FP32, of max |p|).  The right-hand sides hold all modes (white noise),
the null modes among them.  (192, 256, 256) and (96, 256, 512) have more than
2^21 cells, where the other factor of ny goes first.  The last three shapes lie
next to the tables and stay on the general passes.
"""
import numpy as np
import pytest

from oracle import ops
from gpu_util import announce, need_gpu, rel_err, to_np
from test_gpu_fft_pipe import case

pytestmark = pytest.mark.gpu

SHAPES = [(16, 24, 32), (24, 32, 48), (32, 96, 64), (36, 128, 72), (48, 144, 96), (54, 192, 108), (64, 256, 128),
          (72, 72, 144), (96, 64, 192), (108, 48, 216), (128, 36, 256), (144, 108, 288), (192, 48, 384),
          (256, 24, 432), (16, 32, 512), (16, 72, 576), (24, 96, 768), (16, 64, 1024),
          (18, 27, 36), (27, 54, 54), (81, 81, 162), (162, 162, 64), (216, 216, 48), (32, 64, 324), (18, 54, 486),
          (192, 256, 256), (96, 256, 512),
          (24, 32, 972), (24, 243, 48), (2, 32, 48)]


@pytest.mark.parametrize("form", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", SHAPES)
def test_split_solve(shape, form):
    torch, m = need_gpu()
    sc = case(shape, 3)
    announce(f"three-pass solve {form} shape={shape}")
    S = m.Solver(sc, precision=m.FP64 if form == "fp64" else m.FP32_REFINE)
    r = np.random.default_rng(33).standard_normal(shape)
    got = to_np(S.poisson(r))
    again = S._dev(r).clone()
    S.poisson(again, out=again)          # rhs and result may alias
    assert np.array_equal(got, to_np(again))
    S.close()
    ref = ops.poisson_solve(S_round(r, form), sc.spacing)
    err = rel_err(got, ref)
    print(f"[split] {form} {shape} {err:.2e}", flush=True)
    assert err < (1e-11 if form == "fp64" else 1e-5), err


def S_round(r, form):
    return r if form == "fp64" else r.astype(np.float32).astype(np.float64)
