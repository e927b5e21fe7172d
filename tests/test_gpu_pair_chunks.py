"""Stage pairs as the default rule picks them, on the smallest grids that get
them and with a last z chunk shorter than the others, against one kernel per
stage.

Tolerances: those of the stage-pair tests (the two paths evaluate the same
expressions): 1e-12 of the largest value in FP64, 1e-5 in the FP32 form.
"""
import pytest

import scenarios
from gpu_util import announce, need_gpu, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,grid,tol", [
    ("FP64", (64, 128, 162), 1e-12),          # 16 tiles: 15 chunks, the last of 8 planes
    ("FP64", (512, 512, 4), 1e-12),           # one chunk of the least nz
    ("FP64", (192, 96, 64), 1e-12),           # 36 tiles: chunks of 11, the last of 9
    ("FP32_REFINE", (128, 128, 162), 1e-5),   # 32 tiles, two blocks per CU
])
def test_default_pairs_match_single_stages(form, grid, tol):
    torch, m = need_gpu()
    sc = scenarios.room(*grid, dx=0.0390625, n_boxes=3, seed=77) if grid[2] > 8 else \
        scenarios.room(*grid, dx=0.0390625, n_boxes=0, seed=77)
    announce(f"default pairs {form} {grid}")
    out = []
    for mode in (-1, 0):
        S = m.Solver(sc, precision=getattr(m, form))
        S.set_stage_pairs(mode)
        d = S.step(3)
        out.append((S.state(), d))
        S.close()
    for k in ("u", "v", "w", "p", "c"):
        assert rel_err(out[0][0][k], out[1][0][k]) < tol, k
    for k in ("ke", "co2_mass", "cfl_max", "div_l2"):
        assert abs(out[0][1][k] - out[1][1][k]) <= 10 * tol * abs(out[1][1][k]) + (1e-9 if k == "div_l2" else 0.0), k
