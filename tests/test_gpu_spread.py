"""Contact workgroups among the tiles (3D lattices of 4096 tiles and more)
against the oracle's coupled loop: tile counts that are no multiple of 8, in
row and flat tiles, particle counts whose contact groups are one, a few and
many.  Tolerances: FP64 as for the other DEM tests; FP32 the form's 1e-5 of
the largest change of velocity (the contact forces are FP64 in both)."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import gpu_lattice, relerr

pytestmark = pytest.mark.gpu

BOXES = {"row": (64, 67, 241), "flat": (65, 67, 229)}  # 4097 and 4122 tiles


@pytest.mark.parametrize("form", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [5, 130, 1792])
@pytest.mark.parametrize("box", sorted(BOXES))
def test_contacts_among_the_tiles(box, n, form):
    import paper_1901_09745_amd.psclbm as P
    print(f"case: {box} n {n} {form}", flush=True)
    nx, ny, nz = BOXES[box]
    rng = np.random.default_rng(n)
    lat = W.LatticeSpec(q=19, nx=nx, ny=ny, nz=nz, tau=0.8, force=(1e-5, 0, 0))
    # a cubic lattice of spheres that touch along x and y
    ijk = np.array([(i, j, k) for k in range(28) for j in range(8) for i in range(8)][:n], float)
    x = 4.0 + 8.0 * ijk + rng.uniform(-0.05, 0.05, (n, 3))
    u, w = rng.normal(0, 1e-3, (n, 3)), np.zeros((n, 3))
    p = W.Particles(x, u, w, np.full(n, 4.05))
    dem = W.DemSpec(E_p=1e-3, eta_n=0.05, n_sub=1, gamma=1e-5)
    ref, D, pr = oracle.Lattice(lat), oracle.Dem(lat, dem, n), p.copy()
    G, dp = gpu_lattice(lat, p, form), P.DeviceParticles.from_host(p)
    for _ in range(2):
        F, T = ref.step(pr)
        D.step(pr, F, T)
    G.coupled_step(P.make_dem_params(dem), dp, 2)
    G.sync()
    du = np.abs(pr.u - p.u).max()
    assert du > 1e-7  # the contacts act
    tol = 1e-11 if form == "fp64" else 1e-5 * du
    assert np.abs(dp.u.cpu().numpy() - pr.u).max() < tol
    assert np.abs(dp.x.cpu().numpy() - pr.x).max() < 2 * tol + 1e-12  # two steps of it
    assert relerr(G.get_f().cpu().numpy(), ref.f) < (1e-12 if form == "fp64" else 1e-5)
