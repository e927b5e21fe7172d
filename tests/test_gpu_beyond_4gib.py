"""Whole steps on fields of 4 GiB and more, which the byte offsets of the
register-ring kernels do not reach: the stage pairs, the ring filter and the
ring correction have to give way to the other kernels there.  At exactly 4 GiB
(2^29 cells in FP64) only the last cell is out of reach.

A state that repeats along z stays so: every copy of the short period must end
as the same steps on a grid of one period do (its Fourier modes are the same,
at multiples of the number of copies).

Tolerances: FP64 1e-10 of the largest value, the whole-step bar of the parity
tests; the FP32 form rel L2 1e-5, the bar between two launches of the same
expressions.
"""
from types import SimpleNamespace

import pytest

from gpu_util import announce, need_gpu

pytestmark = pytest.mark.gpu
FIELDS = ("u", "v", "w", "p", "c")


def case(torch, shape, copies):
    nz, ny, nx = shape
    gen = torch.Generator(device="cuda").manual_seed(51)
    beta = torch.ones(shape, dtype=torch.uint8, device="cuda")
    beta[nz // 4: nz // 2, ny // 3: ny // 3 + 40, -20:] = 0      # a box, to the seam
    beta[-3:, 5:25, 70:140] = 0                                  # and one across the copies' seam
    beta[:2, 5:25, 70:140] = 0
    forced = torch.zeros(shape, dtype=torch.bool, device="cuda")
    forced[:, ny - 40:, :6] = True
    idx = (forced & (beta == 1)).flatten().nonzero().flatten()

    def field(scale, mean=0.0):
        f = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)
        return (mean + scale * f) * beta

    rep = lambda t: t.repeat(copies, 1, 1)
    k = idx.numel() * copies
    n = nz * ny * nx
    full = lambda v: torch.full((k,), v, dtype=torch.float64)
    return SimpleNamespace(
        nx=nx, ny=ny, nz=nz * copies, lx=nx * 0.05, ly=ny * 0.045, lz=nz * copies * 0.055, nu=1.3e-3, alpha_c=0.9e-3,
        tau_f=0.07, body=(0.01, -0.02, 0.005), cfl=0.3, dt_fixed=2e-4, u_ref=1.0, n_piter=2, filter=True,
        beta=rep(beta), forced_idx=torch.cat([idx + q * n for q in range(copies)]), forced_S=full(0.6),
        forced_uset=torch.full((k, 3), 0.3, dtype=torch.float64), forced_cset=full(400.0), room_mask=None,
        u=rep(field(0.3)), v=rep(field(0.3)), w=rep(field(0.3)), p=rep(field(0.0)), c=rep(field(50.0, 400.0)))


@pytest.mark.parametrize("form,shape,copies", [
    ("FP64", (64, 1024, 1024), 8),            # 2^29 cells
    ("FP64", (48, 972, 972), 12),             # a little more, tiles that do not divide the grid
    ("FP32_REFINE", (72, 1296, 972), 12),     # more than 2^30 cells
])
def test_step_of_repeated_state(form, shape, copies):
    torch, m = need_gpu()
    if torch.cuda.mem_get_info()[1] < 200e9:
        pytest.skip("needs 150 GB of device memory")
    announce(f"repeated state {form} {shape} x {copies}")

    def run(n):
        S = m.Solver(case(torch, shape, n), precision=getattr(m, form))
        S.step(1, diag=False)
        S.set_stage_pairs(1)         # wherever supported
        d = S.step(1)
        f = {k: getattr(S, k) for k in FIELDS}
        S.close()
        return f, d

    one, d1 = run(1)
    many, dn = run(copies)
    for k in FIELDS:
        ref = one[k].double()
        if form != "FP64" and k == "p":
            continue
        for q, got in enumerate(many[k].reshape(copies, *shape)):
            diff = got.double() - ref
            if form == "FP64":
                err, tol = float(diff.abs().max() / ref.abs().max()), 1e-10
            else:
                err, tol = float(diff.norm() / ref.norm()), 1e-5
            assert err < tol, (k, q, err)
    tol = 1e-10 if form == "FP64" else 1e-5
    for k in ("ke", "co2_mass"):
        assert abs(dn[k] - copies * d1[k]) < tol * abs(dn[k]), k
    assert abs(dn["cfl_max"] - d1["cfl_max"]) < tol * d1["cfl_max"]
    del one, many
    torch.cuda.empty_cache()
