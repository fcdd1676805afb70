"""Fields and canonical state read back from every storage form at both
streaming parities, on lattices whose size is no multiple of a workgroup.

Tolerance: both sides sum the same Q stored values (at most one each, FP64)
in FP64, 19 roundings of 2^-53 of a sum of about one, then one division."""
import numpy as np
import pytest

import workloads as W
from helpers import _print_case, gpu_lattice

pytestmark = pytest.mark.gpu

TOL = 2 * 20 * 2.0 ** -53
BOXES = {"d2q9": (9, 67, 13, 1), "d3q19": (19, 9, 7, 13), "one_wave": (9, 3, 2, 1)}


@pytest.mark.parametrize("steps", [0, 1, 2])
@pytest.mark.parametrize("form", ["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("box", sorted(BOXES))
def test_fields_are_the_moments_of_the_state(box, form, steps):
    import torch
    import paper_1901_09745_amd.psclbm as P
    q, nx, ny, nz = BOXES[box]
    F = (3e-4, -2e-4, 0.0 if q == 9 else 1e-4)
    lat = W.LatticeSpec(q=q, nx=nx, ny=ny, nz=nz, tau=0.7, force=F,
                        faces=("periodic",) * 2 + ("bounce_back",) * 2 + ("periodic",) * 2)
    _print_case(test="fields", box=box, form=form, steps=steps)
    G = gpu_lattice(lat, None, form)
    G.set_f(torch.from_numpy(W.random_state(lat, 8)).cuda())
    G.rasterize(None)
    if steps:
        G.step(steps)
    f = G.get_f().cpu().numpy()
    rho, u = (t.cpu().numpy() for t in G.macros())
    E = {9: [(0, 0, 0), (1, 0, 0), (0, 1, 0), (-1, 0, 0), (0, -1, 0), (1, 1, 0), (-1, 1, 0),
             (-1, -1, 0), (1, -1, 0)],
         19: [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1),
              (1, 1, 0), (-1, -1, 0), (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1),
              (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1), (0, -1, 1)]}[q]
    ref = f.sum(0)
    assert np.abs(rho - ref).max() <= TOL
    for a in range(3):
        ju = (np.tensordot(np.array([e[a] for e in E], float), f, (0, 0)) + 0.5 * F[a]) / ref
        assert np.abs(u[..., a] - ju).max() <= TOL
    # either output alone
    only = torch.zeros_like(torch.from_numpy(rho)).cuda()
    P.lbm_get_macros(G.ctx, only, None)
    assert torch.equal(only.cpu(), torch.from_numpy(rho))
    only = torch.zeros(u.shape, dtype=torch.float64, device="cuda")
    P.lbm_get_macros(G.ctx, None, only)
    assert torch.equal(only.cpu(), torch.from_numpy(u))


@pytest.mark.parametrize("n", [1, 43, 86])  # 6 n below, just above and past a workgroup
def test_force_rows_alone_and_together(n):
    import torch
    import paper_1901_09745_amd.psclbm as P
    rng = np.random.default_rng(n)
    lat = W.LatticeSpec(q=9, nx=200, ny=180, tau=0.8, force=(1e-5, 0, 0))
    x = np.array([[10.0 + 18 * (k % 10), 10.0 + 18 * (k // 10), 0.0] for k in range(n)])
    u = np.zeros((n, 3))
    u[:, :2] = rng.normal(0, 1e-2, (n, 2))
    G = gpu_lattice(lat, W.Particles(x, u, np.zeros((n, 3)), np.full(n, 5.0)))
    dp = P.DeviceParticles(x, u, np.zeros((n, 3)), np.full(n, 5.0))
    G.rasterize(dp)
    G.step(1)
    F, T = G.forces()
    # fluid at rest: each disk drags it along its own velocity (Eq. 14)
    assert torch.all((F[:, :2] * dp.u[:, :2]).sum(1) < 0)
    assert torch.all(F[:, 2] == 0) and torch.all(T[:, :2] == 0)
    for k, ref in enumerate((F, T)):
        out = torch.full((n, 3), 7.0, dtype=torch.float64, device="cuda")
        P.particle_forces(G.ctx, *((out, None) if k == 0 else (None, out)))
        assert torch.equal(out, ref)


@pytest.mark.parametrize("chunks", [(1,), (2,), (1, 3, 2)])
@pytest.mark.parametrize("path", ["step", "coupled", "coupled_empty"])
@pytest.mark.parametrize("form", ["fp64", "fp32", "fp16"])
def test_mass_is_the_sum_of_the_state(form, path, chunks):
    """The mass partials that a call's last step forms describe the state it
    leaves.  Tolerance: the sum of the state exactly; the device's is a tree of
    about 40 roundings of deviations below rho0, and one of each population."""
    import math
    import torch
    import paper_1901_09745_amd.psclbm as P
    lat = W.LatticeSpec(q=19, nx=9, ny=17, nz=13, tau=0.7, force=(1e-4, 0, 0),
                        faces=("periodic",) * 2 + ("bounce_back",) * 2 + ("periodic",) * 2)
    n = 0 if path == "coupled_empty" else 1
    x, u = np.full((n, 3), [4.2, 8.3, 6.1]), np.full((n, 3), [0.01, 0.0, 0.02])
    dp = P.DeviceParticles(x, u, np.zeros((n, 3)), np.full(n, 3.0))
    prm = P.make_dem_params(W.DemSpec(E_p=1e-3, eta_n=0.05, n_sub=1, kinematic=True))
    _print_case(test="mass", form=form, path=path, chunks=chunks)
    G = gpu_lattice(lat, W.Particles(x, u, np.zeros((n, 3)), np.full(n, 3.0)), form)
    G.set_f(torch.from_numpy(W.random_state(lat, 8)).cuda())
    G.rasterize(dp)
    for k in chunks:
        if path == "step":
            G.step(k)
        else:
            G.coupled_step(prm, dp, k)
        m = G.mass()
        ref = math.fsum(G.get_f().cpu().numpy().ravel().tolist())
        assert abs(m - ref) <= 64 * 2.0 ** -53 * ref
