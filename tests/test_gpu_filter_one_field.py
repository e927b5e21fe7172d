"""The FP32 filter of one field in chunks of its own (half those of the three
velocity components, the last one shorter): the filter alone against the oracle
and the CO2 mass that the step's filter adds up in those chunks against the sum
over the fields.

Tolerances: 1e-5 of the largest value for the FP32 filter, as in the operator
tests; the mass is a sum of the stored values in FP64, 1e-12.
"""
import numpy as np
import pytest

from oracle import ops
from gpu_util import announce, need_gpu, rel_err, to_np
from test_gpu_parity import make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(162, 144, 192), (512, 128, 64), (216, 108, 216)])
def test_filter_of_one_field(shape):
    torch, m = need_gpu()
    sc = make_case(shape, 13, dt_fixed=2e-4)
    announce(f"one-field filter {shape}")
    S = m.Solver(sc, precision=m.FP32_REFINE)
    assert rel_err(to_np(S.filter(sc.c)), sc.beta * ops.filter6(sc.c, sc.spacing)) < 1e-5
    d = S.step(1)
    c = to_np(S.c)
    S.close()
    mass = float(np.sum(c * sc.beta)) * np.prod(sc.spacing)
    assert abs(d["co2_mass"] - mass) < 1e-12 * abs(mass)
