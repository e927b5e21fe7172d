"""The particle sort at the sizes where its chunk length, its scratch and the
fusing of its scans change (4, 8 or 16 keys per thread up to 2^21, 2^22 and
beyond; all arrays permuted at once up to 2^22; the scan's block totals added up
in the scatter up to 256 scan blocks), against numpy's stable argsort of the
cell index, exactly; and a step across the periodic seam of x against the oracle
(particles in the last cell, whose upper corner wraps).
"""
import numpy as np
import pytest

from oracle import particles as po
from gpu_util import announce, need_gpu, rel_err
from test_gpu_particles import G, RHO_F, RHO_P, setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1025, (1 << 21) - 1, (1 << 21) + 1, (1 << 22) + 1, (1 << 24) + (1 << 20) + 3])
def test_sort_sizes(n):
    torch, m, sc, S, box, pos, vel, diam, t = setup(n=8, seed=13)
    announce(f"particles sort n={n}")
    g = torch.Generator(device="cuda").manual_seed(n)
    b = torch.tensor(box, dtype=torch.float64, device="cuda")[:, None]
    p = torch.rand((3, n), dtype=torch.float64, device="cuda", generator=g) * b
    p[:, ::50] = p[:, :1]                      # ties
    v = torch.randn((3, n), dtype=torch.float64, device="cuda", generator=g)
    dm = torch.rand(n, dtype=torch.float64, device="cuda", generator=g) * 1e-5 + 1e-6
    h = [a.cpu().numpy() for a in (p, v, dm)]
    for _ in range(2):                         # the second time on sorted input
        S.particles_sort(p, v, dm)
        idx = [np.floor(h[0][a] / sc.spacing[a]).astype(np.int64) % k for a, k in enumerate((sc.nx, sc.ny, sc.nz))]
        o = np.argsort(idx[0] + sc.nx * (idx[1] + sc.ny * idx[2]), kind="stable")
        h = [h[0][:, o], h[1][:, o], h[2][o]]
        for got, ref in zip((p, v, dm), h):
            assert np.array_equal(got.cpu().numpy(), ref)
    S.close()


def test_step_in_the_last_cells():
    torch, m, sc, S, box, pos, vel, diam, t = setup(n=4096, seed=17)
    announce("particles step, last cells")
    rng = np.random.default_rng(18)
    # x in the last cell, y and z in the last cell for a half each
    pos[0] = (sc.nx - 1 + rng.uniform(0.0, 1.0, pos.shape[1])) * sc.spacing[0]
    pos[1, ::2] = (sc.ny - 1 + 0.5) * sc.spacing[1]
    pos[2, 1::2] = (sc.nz - 1 + 0.25) * sc.spacing[2]
    u = [q.double().cpu().numpy() for q in (S.u, S.v, S.w)]
    rp, rv = po.step(pos, vel, diam, u, sc.spacing, box, sc.nu, RHO_P, RHO_F, G, 1e-3)
    tp, tv, td = t(pos), t(vel), t(diam)
    S.particles_step(tp, tv, td, RHO_P, RHO_F, G, dt=1e-3)
    assert rel_err(tp.cpu().numpy(), rp) < 1e-12
    assert rel_err(tv.cpu().numpy(), rv) < 1e-12
    S.close()
