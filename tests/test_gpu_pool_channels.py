"""2D channels in one pool: their solves go axis by axis in batched launches, one
per transform length where the lengths differ.  Each scenario must end bitwise
equal to its pool of one, which issues its steps directly.
"""
import numpy as np
import pytest

from gpu_util import announce, need_gpu
from test_gpu_parity import make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["FP64", "FP32_REFINE"])
def test_pool_of_channels_of_several_lengths(form):
    torch, m = need_gpu()
    from paper_2204_02107_amd.serving import Pool
    prec = getattr(m, form)
    # two of equal lengths; x and y lengths in which the others differ, one with
    # an odd nx/2 and a last column tile that is not full
    cs = [make_case(shape, seed, dt_fixed=1e-3)
          for shape, seed in (((1, 54, 432), 61), ((1, 54, 432), 62), ((1, 64, 432), 63), ((1, 81, 486), 64),
                              ((1, 192, 1536), 65))]
    steps = 5
    announce(f"pool of channels {form}")
    alone = []
    for c in cs:
        pool = Pool(4 << 30, prec)
        s = pool.admit(c, steps)
        pool.step(steps)
        alone.append(pool.state(s, c.shape))
        pool.close()
    pool = Pool(4 << 30, prec)
    slots = [pool.admit(c, steps) for c in cs]
    assert None not in slots
    pool.step(2)
    pool.step(steps - 2)
    for q, c in enumerate(cs):
        got = pool.state(slots[q], c.shape)
        for k in ("u", "v", "w", "p", "c"):
            assert np.all(np.isfinite(got[k])), (q, k)
            assert np.array_equal(got[k], alone[q][k]), (q, k)
    pool.close()
