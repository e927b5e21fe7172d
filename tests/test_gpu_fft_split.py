"""The FFT solves on register tiles against the oracle's Poisson solve (Section
2.2): the three-pass solve (the y transform split between the x passes and the
z pass) and the axis-by-axis one.

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


# The axis-by-axis solve: every x length and column length of its tables, 2D
# (nz = 1, one column pass) and 3D with y transforms too long to be split.
LINE_SHAPES = [(1, 54, 324), (1, 64, 384), (1, 72, 432), (1, 81, 486), (1, 96, 512), (1, 108, 576), (1, 128, 648),
               (1, 144, 768), (1, 162, 864), (1, 192, 972), (1, 216, 1024), (1, 243, 1152), (1, 256, 1296),
               (1, 288, 1458), (1, 324, 1536), (1, 384, 1728), (1, 432, 1944), (1, 512, 2048), (1, 54, 2304),
               (1, 64, 2592), (1, 54, 2916), (1, 64, 3072), (1, 54, 3456),
               (54, 288, 324), (64, 512, 384), (81, 324, 432), (96, 432, 512), (243, 54, 972), (128, 384, 324)]


@pytest.mark.parametrize("form", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", SHAPES + LINE_SHAPES)
def test_split_solve(shape, form):
    torch, m = need_gpu()
    sc = case(shape, 3)
    announce(f"register-tile solve {form} shape={shape}")
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
