"""The lattice step, solid fractions and adjoint on lattices whose rows do
not fill a wave: rows of 1 to 129 cells around the wave's 64, rows that share
a wave, planes shorter than a workgroup, with periodic, resting and moving
walls, and with particles that several rows and tiles see through the
periodic wrap.  FP64 against the oracle (1e-12, as everywhere); the reduced
forms against an FP64 step from the very state they held (one step is fewer
than 64 FP32 roundings of the largest deviation; FP16 storage adds 2^-11)."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import _print_case, force_scale, gpu_lattice, relerr

pytestmark = pytest.mark.gpu

PER, BB, MW = W.PERIODIC, W.BOUNCE_BACK, W.MOVING_WALL
FACES = {"periodic": (PER,) * 6, "walls_x": (BB, MW) + (PER,) * 4,
         "walls_y": (PER, PER, MW, BB, PER, PER)}
# q, nx, ny, nz, particles
SIZES = [(9, 1, 5, 1, 0), (9, 2, 3, 1, 0), (9, 7, 130, 1, 0), (9, 24, 70, 1, 2),
         (9, 63, 30, 1, 2), (9, 64, 30, 1, 2), (9, 65, 31, 1, 2), (9, 100, 50, 1, 4),
         (9, 129, 33, 1, 3), (19, 1, 2, 4, 0), (19, 3, 70, 2, 0), (19, 18, 19, 17, 2),
         (19, 33, 18, 20, 2), (19, 65, 17, 18, 3), (19, 80, 20, 16, 4), (19, 130, 16, 16, 4)]


def _case(q, nx, ny, nz, n, faces):
    f = FACES[faces]
    lat = W.LatticeSpec(q=q, nx=nx, ny=ny, nz=nz, tau=0.7, force=(2e-5, -1e-5, 0), faces=f,
                        face_u=((0, 0, 0), (0, 0.01, 0), (0.012, 0, 0)) + ((0, 0, 0),) * 3)
    if n == 0:
        return lat, None
    rng = np.random.default_rng(nx + 7 * ny)
    D = 2 if q == 9 else 3
    L = np.array([nx, ny, nz])
    x, u, w = np.zeros((n, 3)), np.zeros((n, 3)), np.zeros((n, 3))
    r = rng.uniform(2.5, 4.0, n)
    for a in range(D):
        edge = 0.0 if f[2 * a] == PER else 1.0
        x[:, a] = rng.uniform(edge, L[a] - 1 - edge, n)
        u[:, a] = rng.normal(0, 5e-3, n)
    x[0, 0] = nx - 0.3 if f[0] == PER else x[0, 0]  # covers cells on both sides of the wrap
    x[0, 1] = 0.2 if f[2] == PER else x[0, 1]
    w[:, 0 if D == 3 else 2:] = rng.normal(0, 1e-3, (n, 3 if D == 3 else 1))
    return lat, W.Particles(x, u, w, r)


@pytest.mark.parametrize("faces", sorted(FACES))
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "x".join(map(str, s)))
def test_ragged_step_and_fractions(size, faces):
    import torch
    import paper_1901_09745_amd.psclbm as P
    q, nx, ny, nz, n = size
    lat, p = _case(*size, faces)
    _print_case(test="ragged", size=size, faces=faces)
    f0 = W.random_state(lat, 9, amp=1e-2)
    ref = oracle.Lattice(lat, f0)
    G = gpu_lattice(lat, p)
    G.set_f(torch.from_numpy(f0).cuda())
    dp = None if p is None else P.DeviceParticles.from_host(p)
    G.rasterize(dp)
    if p is not None:
        eps, ids, seps = G.solid_fraction()
        _, rid, reps, tot = oracle.rasterize(lat, p.x, p.r)
        assert np.array_equal(ids.cpu().numpy().reshape(-1, 4), np.asarray(rid)[:, :4])
        assert np.abs(seps.cpu().numpy().reshape(-1, 4) - np.asarray(reps)[:, :4]).max() < 1e-13
    for _ in range(3):
        before = ref.f.copy()
        F, T = ref.step(p)
        G.step(1)
    G.sync()
    assert relerr(G.get_f().cpu().numpy(), ref.f) < 1e-12
    if p is not None:
        Fg, _ = G.forces()
        assert np.all(np.abs(Fg.cpu().numpy() - F).max(1) <= 1e-12 * force_scale(lat, before, p) + 1e-300)
    # the reduced forms, both parities
    w = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4 if q == 9 else
                 [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12).reshape(-1, 1, 1, 1)
    H = gpu_lattice(lat, p)
    H.rasterize(dp)
    for form, store in (("fp32", 0.0), ("fp16", 2.0 ** -11)):
        R = gpu_lattice(lat, p, form)
        R.set_f(torch.from_numpy(f0).cuda())
        R.rasterize(dp)
        for _ in range(2):
            held = R.get_f()
            H.set_f(held)
            H.step(1)
            R.step(1)
            a, b = H.get_f().cpu().numpy(), R.get_f().cpu().numpy()
            size_ = max(np.abs(a - w).max(), np.abs(held.cpu().numpy() - w).max())
            assert np.abs(a - b).max() <= (64 * 2.0 ** -24 + store) * size_
        R.sync()


@pytest.mark.parametrize("size", [s for s in SIZES if s[4]], ids=lambda s: "x".join(map(str, s)))
def test_ragged_adjoint_step(size):
    """One adjoint step against the directional derivative of the oracle's
    step (central differences, h = 1e-6: the step is analytic in f, u and
    omega, so O(h^2) is below the rounding 1e-16 / h of the differences)."""
    import torch
    import paper_1901_09745_amd.psclbm as P
    lat, p = _case(*size, "periodic")
    _print_case(test="ragged adjoint", size=size)
    rng = np.random.default_rng(4)
    f0 = W.random_state(lat, 10, amp=1e-2)
    lam, gF = rng.normal(size=f0.shape), rng.normal(size=(p.n, 3))
    gT = rng.normal(size=(p.n, 3))
    if lat.q == 9:
        gF[:, 2] = 0
        gT[:, :2] = 0
    G = gpu_lattice(lat, p)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    G.rasterize(P.DeviceParticles.from_host(p))
    out = torch.empty(f0.shape, dtype=torch.float64, device="cuda")
    gx, gu, gw = (torch.zeros((p.n, 3), dtype=torch.float64, device="cuda") for _ in range(3))
    P.lbm_step_adjoint(G.ctx, t(f0), t(lam), out, t(gF), t(gT), gx, gu, gw, None)
    G.sync()
    df, du, dw = rng.normal(size=f0.shape) * 1e-2, rng.normal(size=(p.n, 3)), rng.normal(size=(p.n, 3))
    if lat.q == 9:
        du[:, 2] = 0
        dw[:, :2] = 0

    def J(h):
        L = oracle.Lattice(lat, f0 + h * df)
        F, T = L.step(W.Particles(p.x, p.u + h * du, p.omega + h * dw, p.r))
        return np.array([(L.f * lam).sum(), (F * gF).sum(), (T * gT).sum()])

    h = 1e-6
    num = ((J(h) - J(-h)) / (2 * h)).sum()
    got = float((out.cpu().numpy() * df).sum() + (gu.cpu().numpy() * du).sum() +
                (gw.cpu().numpy() * dw).sum())
    # the differences round at eps times the sizes of the three sums, over h
    size_ = np.abs(f0 * lam).sum() + 100.0
    assert abs(got - num) <= 4 * 2.0 ** -53 * size_ / h + 1e-9 * abs(num)
    # recomputed states are the step's
    ring = torch.empty((2,) + f0.shape, dtype=torch.float64, device="cuda")
    P.lbm_recompute(G.ctx, t(f0), 2, ring)
    ref = oracle.Lattice(lat, f0)
    for k in range(2):
        ref.step(p)
        assert relerr(ring[k].cpu().numpy(), ref.f) < 1e-12
