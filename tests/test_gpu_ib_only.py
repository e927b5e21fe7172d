"""Projection on grids of 2^23 cells or more, where the immersed-boundary
iterates are written only where the next iterate's right-hand side reads them
(Section 2.2): against the oracle's iteration from a random warm start, with
boxes placed anywhere (also across the periodic seams), for the three-pass solve
and the axis-by-axis one.  FP64 bar: the projection bar of the parity tests,
1e-11 of the largest value, four solves deep.
"""
import numpy as np
import pytest

import scenarios
from oracle.step import Oracle
from gpu_util import announce, need_gpu, rel_err, to_np
from test_gpu_parity import make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(128, 256, 256), (54, 512, 324)])
def test_projection_with_partly_written_iterates(shape):
    torch, m = need_gpu()
    sc = make_case(shape, 41, forced=False)
    sc.beta = scenarios.random_beta(shape, 7, n_boxes=5, max_size=20)
    b = sc.beta.astype(np.float64)
    sc.u, sc.v, sc.w = sc.u * b, sc.v * b, sc.w * b
    announce(f"projection, partly written iterates, shape={shape}")
    S = m.Solver(sc)
    f = [S._dev(a).clone() for a in (sc.u, sc.v, sc.w)]
    S.project(*f)
    got = [to_np(t) for t in f] + [to_np(S.p)]
    S.close()
    u, p = Oracle.from_scenario(sc).project([sc.u, sc.v, sc.w], sc.p)
    for g, r, name in zip(got, list(u) + [p], "uvwp"):
        err = rel_err(g, r)
        assert err < 1e-11, (name, err)
