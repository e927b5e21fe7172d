"""Tiled kernels on grids that their tiles do not divide: the last tile of a row
starts early and leaves the cells it shares with the tile before it to that one.
Widths of one tile and a little more, of nearly two, and row counts of the
least, one more and odd remainders, for the stage pairs (64 x 8), the LDS
stages and filter (64 x 4 to 64 x 16) and, from 2^21 cells on, the ring filter
and correction (64 x 16), the latter also in place.

Tolerances: those of the stage-pair and whole-step tests: FP64 1e-10 of the
largest value against the oracle and 1e-12 between two launches of the same
expressions; the FP32 form rel L2 1e-4 against the oracle and 1e-5 between.
"""
import numpy as np
import pytest

from oracle.step import Oracle
from gpu_util import announce, need_gpu, rel_err, to_np
from test_gpu_parity import make_case

pytestmark = pytest.mark.gpu
FIELDS = ("u", "v", "w", "p", "c")


def rel_l2(got, ref):
    return float(np.sqrt(np.sum((got - ref) ** 2) / max(np.sum(ref ** 2), 1e-300)))


def run(m, sc, form, mode, steps):
    S = m.Solver(sc, precision=getattr(m, form))
    S.set_stage_pairs(mode)
    d = S.step(steps)
    st = S.state()
    S.close()
    return st, d


@pytest.mark.parametrize("form", ["FP64", "FP32_REFINE"])
@pytest.mark.parametrize("shape", [(6, 8, 72), (9, 9, 108), (16, 12, 96), (4, 18, 162), (12, 27, 64), (6, 24, 216)])
def test_pairs_and_stages(shape, form):
    torch, m = need_gpu()
    announce(f"part tiles {shape} {form}")
    sc = make_case(shape, 31, dt_fixed=2e-4)
    steps = 3
    pairs, d1 = run(m, sc, form, 1, steps)
    single, d0 = run(m, sc, form, 0, steps)
    O = Oracle.from_scenario(sc)
    st, diags = O.run(Oracle.state_from_scenario(sc), steps)
    for k in FIELDS:
        ref = getattr(st, k)
        if form == "FP64":
            assert rel_err(pairs[k], single[k]) < 1e-12, k
            assert rel_err(pairs[k], ref) < 1e-10, k
        else:
            assert rel_l2(pairs[k], single[k]) < 1e-5, k
            if k != "p":
                assert rel_l2(pairs[k], ref) < 1e-4, k
    tol = 1e-10 if form == "FP64" else 1e-4
    for k in ("ke", "co2_mass", "co2_room_mean", "cfl_max"):
        assert abs(d1[k] - diags[-1][k]) <= tol * abs(diags[-1][k]), k
        assert abs(d0[k] - diags[-1][k]) <= tol * abs(diags[-1][k]), k


@pytest.mark.parametrize("shape", [(144, 54, 288)])
def test_large_step_and_project(shape):
    torch, m = need_gpu()
    announce(f"part tiles, step and projection {shape}")
    sc = make_case(shape, 33, dt_fixed=2e-4)
    O = Oracle.from_scenario(sc)
    st, diags = O.run(Oracle.state_from_scenario(sc), 1)
    for form, tol in (("FP64", 1e-10), ("FP32_REFINE", 1e-4)):
        got, d = run(m, sc, form, -1, 1)
        for k in FIELDS:
            if form == "FP64":
                assert rel_err(got[k], getattr(st, k)) < tol, k
            elif k != "p":
                assert rel_l2(got[k], getattr(st, k)) < tol, k
        for k in ("ke", "co2_mass", "co2_room_mean", "cfl_max"):
            assert abs(d[k] - diags[-1][k]) <= tol * abs(diags[-1][k]), (form, k)
    S = m.Solver(sc)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (sc.u, sc.v, sc.w)]
    S.project(*dev)
    ref, _ = O.project([sc.u, sc.v, sc.w], sc.p)[:2]
    for a in range(3):
        assert rel_err(to_np(dev[a]), ref[a]) < 1e-10, a
    S.close()
