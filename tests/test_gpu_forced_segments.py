"""The lookup of a forced cell's entry through 64-cell segments, at the places
where it can go wrong: the first and the last cell, a segment that is forced
whole, one with a single cell, neighbouring segments with gaps, a last segment
that the grid does not fill, and every cell forced.

Each entry carries its own S, u_set and c_set, so that a wrong entry shows.
Tolerances: those of the right-hand-side tests, FP64 1e-12 and FP32 1e-5 of the
largest value (the expressions are the oracle's, only the lookup differs).
"""
import numpy as np
import pytest

from oracle.step import Oracle
from gpu_util import announce, need_gpu, rel_err, to_np
from test_gpu_parity import make_case

pytestmark = pytest.mark.gpu


def cells(kind, n, rng):
    if kind == "ends":
        return np.array([0, n - 1])
    if kind == "all":
        return np.arange(n)
    pick = [np.arange(64, 128), [63 + 128], [256], [319], [320 + 17, 320 + 18], rng.choice(np.arange(448, n), 40)]
    return np.unique(np.concatenate([np.asarray(p, np.int64) for p in pick]))


@pytest.mark.parametrize("form", ["FP64", "FP32_REFINE"])
@pytest.mark.parametrize("shape", [(12, 9, 18), (27, 3, 18)])
@pytest.mark.parametrize("kind", ["ends", "mixed", "all"])
def test_forced_entries(kind, shape, form):
    torch, m = need_gpu()
    announce(f"forced segments {kind} {shape} {form}")
    rng = np.random.default_rng(7)
    sc = make_case(shape, 5)
    n = int(np.prod(shape))
    idx = cells(kind, n, rng)
    sc.forced_idx = idx.astype(np.int64)
    sc.forced_S = rng.uniform(0.2, 1.0, idx.size)
    sc.forced_uset = rng.uniform(-1.0, 1.0, (idx.size, 3))
    sc.forced_cset = rng.uniform(300.0, 900.0, idx.size)
    tol = 1e-12 if form == "FP64" else 1e-5
    S = m.Solver(sc, precision=getattr(m, form))
    O = Oracle.from_scenario(sc)
    got = [to_np(t) for t in S.momentum_rhs(sc.u, sc.v, sc.w)]
    ref = O.F([sc.u, sc.v, sc.w])
    for a in range(3):
        assert rel_err(got[a], ref[a]) < tol, a
    assert rel_err(to_np(S.scalar_rhs(sc.c, sc.u, sc.v, sc.w)), O.G(sc.c, [sc.u, sc.v, sc.w])) < tol
    S.close()
