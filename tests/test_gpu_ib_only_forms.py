"""Partly written immersed-boundary iterates (grids of 2^23 cells or more) in
the FP32 form, whose refinement residual reads the last such iterate as well,
and on lines of more than 1024 cells, whose segments are wider than 16 cells:
the projection against the oracle's from a random warm start.

Tolerances: FP64 1e-11 of the largest value, the projection bar of the parity
tests; the FP32 form 1e-5, the bar of its operators.  The warm start is of size
one and stays in every cell that an iterate leaves out, so a cell read without
being written shows by orders of magnitude more.
"""
import numpy as np
import pytest

import scenarios
from oracle.step import Oracle
from gpu_util import announce, need_gpu, rel_err, to_np
from test_gpu_parity import make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,shape", [
    ("FP32_REFINE", (128, 256, 256)),     # three passes
    ("FP32_REFINE", (54, 512, 324)),      # axis by axis
    ("FP64", (54, 128, 1296)),            # segments of 32 cells
    ("FP32_REFINE", (54, 128, 1296)),
])
def test_projection_with_partly_written_iterates(form, shape):
    torch, m = need_gpu()
    sc = make_case(shape, 43, forced=False)
    sc.beta = scenarios.random_beta(shape, 8, n_boxes=5, max_size=20)
    b = sc.beta.astype(np.float64)
    sc.u, sc.v, sc.w = sc.u * b, sc.v * b, sc.w * b
    announce(f"projection, partly written iterates, {form} {shape}")
    S = m.Solver(sc, precision=getattr(m, form))
    f = [S._dev(a).clone() for a in (sc.u, sc.v, sc.w)]
    S.project(*f)
    got = [to_np(t) for t in f] + [to_np(S.p)]
    S.close()
    u, p = Oracle.from_scenario(sc).project([sc.u, sc.v, sc.w], sc.p)
    tol = 1e-11 if form == "FP64" else 1e-5
    for g, r, name in zip(got, list(u) + [p], "uvwp"):
        err = rel_err(g, r)
        assert err < tol, (name, err)
