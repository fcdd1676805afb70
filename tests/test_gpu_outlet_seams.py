"""x outlets in flat tiles against the oracle, forward (both streaming
parities, and recomputed states) and adjoint: a wave may end at x = 0, whose
neighbour is then in the next wave, or start at x = nx - 1.  FP64 1e-12, as
everywhere; the adjoint against the directional derivative of the oracle's
step in the state and the face velocities (central differences, h = 1e-6,
whose rounding is eps times the size of the sum over h)."""
import dataclasses

import numpy as np
import pytest

import oracle
import workloads as W
from helpers import _print_case, gpu_lattice, relerr

pytestmark = pytest.mark.gpu

IN, OUT, PER, BB = W.INLET_EQ, W.OUTLET_EQ, W.PERIODIC, W.BOUNCE_BACK
# 65 y and 67 y reach 63 mod 64 (x = 0 in a last lane) at y = 63 and 21, 66 + 67 y is 0
# (x = nx - 1 in a first lane) at y = 42; x = 64 is alone in its row's second segment
BOXES = {
    "3d_65": (19, 65, 66, 4, (OUT, OUT, OUT, IN, PER, PER)),
    "3d_67": (19, 67, 45, 5, (OUT, OUT, OUT, OUT, BB, OUT)),
    "3d_3": (19, 3, 70, 4, (OUT, OUT, OUT, OUT, PER, PER)),
    "3d_inlet_67": (19, 67, 45, 5, (IN, OUT, OUT, BB, PER, PER)),
    "2d_67": (9, 67, 45, 1, (OUT, OUT, OUT, IN, PER, PER)),
}


def _case(box):
    q, nx, ny, nz, faces = BOXES[box]
    fu = tuple((0.02 * (f == IN), 0.001 * k * (f == IN), 0.0) for k, f in enumerate(faces))
    return W.LatticeSpec(q=q, nx=nx, ny=ny, nz=nz, tau=0.7, force=(1e-5, -2e-6, 0), faces=faces,
                         face_u=fu)


@pytest.mark.parametrize("box", sorted(BOXES))
def test_outlet_seams_forward(box):
    import torch
    import paper_1901_09745_amd.psclbm as P
    lat = _case(box)
    _print_case(test="outlet seams", box=box)
    f0 = W.random_state(lat, 5, amp=1e-2)
    ref = oracle.Lattice(lat, f0)
    G = gpu_lattice(lat, None)
    G.set_f(torch.from_numpy(f0).cuda())
    G.rasterize(None)
    ring = torch.empty((3,) + f0.shape, dtype=torch.float64, device="cuda")
    P.lbm_recompute(G.ctx, torch.from_numpy(f0).cuda(), 3, ring)
    for k in range(3):
        ref.step(None)
        G.step(1)
        assert relerr(G.get_f().cpu().numpy(), ref.f) < 1e-12
        assert relerr(ring[k].cpu().numpy(), ref.f) < 1e-12
    G.sync()


@pytest.mark.parametrize("box", sorted(BOXES))
def test_outlet_seams_adjoint(box):
    import torch
    import paper_1901_09745_amd.psclbm as P
    lat = _case(box)
    _print_case(test="outlet seams adjoint", box=box)
    rng = np.random.default_rng(6)
    f0 = W.random_state(lat, 8, amp=1e-2)
    lam, df = rng.normal(size=f0.shape), rng.normal(size=f0.shape) * 1e-2
    dv = rng.normal(size=(6, 3)) * np.array([[float(f == IN)] for f in lat.faces])
    if lat.q == 9:
        dv[:, 2] = 0
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    G = gpu_lattice(lat, None)
    G.rasterize(None)
    out = torch.empty(f0.shape, dtype=torch.float64, device="cuda")
    gface = torch.zeros((6, 3), dtype=torch.float64, device="cuda")
    P.lbm_step_adjoint(G.ctx, t(f0), t(lam), out, None, None, None, None, None, gface)
    G.sync()

    def J(h):
        fu = tuple(tuple(np.asarray(v) + h * d) for v, d in zip(lat.face_u, dv))
        L = oracle.Lattice(dataclasses.replace(lat, face_u=fu), f0 + h * df)
        L.step(None)
        return (L.f * lam).sum()

    h = 1e-6
    num = (J(h) - J(-h)) / (2 * h)
    got = float((out.cpu().numpy() * df).sum() + (gface.cpu().numpy() * dv).sum())
    assert abs(got - num) <= 4 * 2.0 ** -53 * np.abs(f0 * lam).sum() / h + 1e-9 * abs(num)
    # every cell by itself, at the waves' edges among them: a direction in one
    # population of the neighbours of the x outlets
    x = [c for c, f in ((1, lat.faces[0]), (lat.nx - 2, lat.faces[1])) if f == OUT]
    g = out.cpu().numpy()
    for c in x:
        for y in range(0, lat.ny, 1 if lat.ny < 50 else 3):
            e = np.zeros_like(f0)
            e[1, 0, y, c] = 1e-2
            Jp, Jm = ((oracle.Lattice(lat, f0 + s * h * e)) for s in (1, -1))
            Jp.step(None)
            Jm.step(None)
            d = ((Jp.f - Jm.f) * lam).sum() / (2 * h)
            # (the difference's terms away from the cell cancel exactly)
            assert abs(1e-2 * g[1, 0, y, c] - d) <= 4 * 2.0 ** -53 * 200 / h + 1e-9 * abs(d)
