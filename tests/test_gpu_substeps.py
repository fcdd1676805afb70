"""coupled_step with DEM sub-steps, whose kernels bin the particles for each
other, against the oracle's coupled loop: every kind of motion, one to three
sub-steps, several calls (each starts its own rasterisation), particles that
cross a periodic face.  Tolerances as for the other DEM tests: positions
1e-9, velocities and spins 1e-11 (contact sums in other orders)."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import gpu_lattice, relerr
from test_gpu_friction import _dense_2d, _walled_3d

pytestmark = pytest.mark.gpu

MOTION = {
    "jkr": dict(gamma=1e-5),
    "hertz": dict(gamma=0.0),
    "friction": dict(gamma=1e-5, k_t=1e-3, eta_t=0.02, mu_f=0.3, theta_r=0.02),
    "prescribed": dict(kinematic=True),
}


@pytest.mark.parametrize("n_sub,calls", [(1, (3, 4)), (2, (1, 1, 5)), (3, (7,))])
@pytest.mark.parametrize("motion", sorted(MOTION))
@pytest.mark.parametrize("box", ["2d", "3d"])
def test_substeps_match_oracle(box, motion, n_sub, calls):
    import paper_1901_09745_amd.psclbm as P
    print(f"case: {box} {motion} n_sub {n_sub} calls {calls}", flush=True)
    lat, p = _dense_2d() if box == "2d" else _walled_3d()
    p.u[:, :2] *= 20.0  # fast enough to touch, slide and cross faces within the run
    p.x[0, 1] = lat.ny - 0.01
    p.u[0, 1] = 0.03
    dem = W.DemSpec(E_p=1e-3, eta_n=0.05, n_sub=n_sub, **MOTION[motion])
    ref, D, pr = oracle.Lattice(lat), oracle.Dem(lat, dem, p.n), p.copy()
    G, dp, prm = gpu_lattice(lat, p), P.DeviceParticles.from_host(p), P.make_dem_params(dem)
    for k in calls:
        for _ in range(k):
            F, T = ref.step(pr)
            D.step(pr, F, T)
        G.coupled_step(prm, dp, k)
        G.sync()
        assert relerr(G.get_f().cpu().numpy(), ref.f) < 1e-12
        assert np.abs(dp.x.cpu().numpy() - pr.x).max() < 1e-9
        assert np.abs(dp.u.cpu().numpy() - pr.u).max() < 1e-11
        assert np.abs(dp.omega.cpu().numpy() - pr.omega).max() < 1e-11
    assert pr.x[0, 1] < 1.0  # it crossed
