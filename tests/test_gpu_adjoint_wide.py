"""lbm_step_adjoint where one direction's FP64 array is 4 GiB or more (a
reduced form of 2^29 cells or more): a state and a sensitivity that repeat
every 16 rows of a periodic lattice give the small lattice's sensitivity,
repeated.

Tolerance: each value is a sum of fewer than 64 products no larger than 20
times the largest sensitivity, rounded in another order at most."""
import pytest

import workloads as W
from helpers import _print_case

pytestmark = pytest.mark.gpu

ROWS = 16


@pytest.mark.parametrize("nx", [8192, 70])  # row tiles, flat tiles
def test_adjoint_beyond_32_bit_offsets(nx):
    import torch
    import paper_1901_09745_amd.psclbm as P
    rep = 2 ** 29 // (nx * ROWS) + 3
    ny = rep * ROWS
    assert nx * ny * 8 > 2 ** 32
    need = 9 * nx * ny * (3 * 8 + 4) * 1.15
    if torch.cuda.mem_get_info()[0] < need:
        pytest.skip("needs %.0f GB of device memory" % (need / 1e9))
    _print_case(test="adjoint beyond 4 GiB", nx=nx, ny=ny)

    def adjoint(form, rows, f, lam, out):
        lat = W.LatticeSpec(q=9, nx=nx, ny=rows, tau=0.7, force=(1e-5, -2e-5, 0.0))
        G = P.Lattice(lat, form, max_particles=1, max_radius=1000.0)  # (few DEM bins)
        G.rasterize(None)
        P.lbm_step_adjoint(G.ctx, f, lam, out, None, None, None, None, None, None)
        G.sync()

    gen = torch.Generator(device="cuda").manual_seed(5)
    new = lambda: torch.randn((9, ROWS, nx), dtype=torch.float64, device="cuda", generator=gen)  # noqa: E731
    w = torch.tensor([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4, dtype=torch.float64, device="cuda")
    f, lam = w[:, None, None] * (1 + 0.05 * new()), new()
    small = torch.empty_like(f)
    adjoint("fp64", ROWS, f, lam, small)

    big = lambda t: torch.empty((9, rep, ROWS, nx), dtype=torch.float64, device="cuda").copy_(t[:, None])  # noqa: E731
    bf, blam = big(f), big(lam)
    out = torch.full_like(bf, float("nan"))
    adjoint("fp32", ny, bf, blam, out)
    tol = 64 * 2.0 ** -53 * 20 * float(lam.abs().max())
    for i in range(9):
        err = float((out[i] - small[i]).abs_().max())
        assert err <= tol, (i, err)
    del bf, blam, out
    torch.cuda.empty_cache()
