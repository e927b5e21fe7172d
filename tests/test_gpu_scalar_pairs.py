"""The scalar's stage pairs where no filter follows them (their result is then
copied to c): a scalar step alone and a step with the filter off, on grids that
the tile divides and that it does not, with the copy's last block whole, short
and of one value.

Tolerances: those of the scalar step's test, 1e-12 (FP64) and 1e-5 (FP32 form)
of the largest value, and 1e-10 / 1e-4 for a whole step.
"""
import pytest

from oracle.step import Oracle
from gpu_util import announce, need_gpu, rel_err, to_np
from test_gpu_parity import make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,tol", [("FP64", 1e-12), ("FP32_REFINE", 1e-5)])
@pytest.mark.parametrize("shape", [(8, 16, 64), (9, 9, 108), (3, 27, 162), (1, 8, 72)])
def test_scalar_step_in_pairs(shape, form, tol):
    torch, m = need_gpu()
    announce(f"scalar pairs {shape} {form}")
    sc = make_case(shape, 12)
    S = m.Solver(sc, precision=getattr(m, form))
    S.set_stage_pairs(1)
    S.scalar_step(0.01)
    ref = Oracle.from_scenario(sc).rk4_scalar(sc.c, [sc.u, sc.v, sc.w], 0.01)
    assert rel_err(to_np(S.c), ref) < tol
    S.close()


@pytest.mark.parametrize("form,tol", [("FP64", 1e-10), ("FP32_REFINE", 1e-4)])
def test_step_without_filter(form, tol):
    torch, m = need_gpu()
    announce(f"scalar pairs, no filter {form}")
    sc = make_case((9, 9, 108), 14, filt=False, dt_fixed=2e-4)
    O = Oracle.from_scenario(sc)
    st, diags = O.run(Oracle.state_from_scenario(sc), 2)
    S = m.Solver(sc, precision=getattr(m, form))
    S.set_stage_pairs(1)
    d = S.step(2)
    assert rel_err(S.state()["c"], st.c) < tol
    for k in ("co2_mass", "co2_room_mean"):
        assert abs(d[k] - diags[-1][k]) <= tol * abs(diags[-1][k]), k
    S.close()
