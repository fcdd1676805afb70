"""Outlet velocities read before the step (faces whose neighbour is in
another wave), in every storage form and streaming parity: a step of the form
against a step of the FP64 form from the very state the form held.

Tolerance: the two start from the same values, so they differ by the form's
arithmetic and the storage of its result.  One step is a chain of fewer than
64 FP32 roundings of values no larger than the largest deviation |f - w rho0|
of either state (2^-24 each); FP16 storage rounds h = g / w once, 2^-11 |h|."""
import numpy as np
import pytest

import workloads as W
from helpers import _print_case, gpu_lattice

pytestmark = pytest.mark.gpu

IN, OUT, PER = W.INLET_EQ, W.OUTLET_EQ, W.PERIODIC
BOXES = {
    # y and z outlets on faces of unequal size; x = nx - 1 in the neighbour's wave
    "d3q19": (19, 37, 11, 6, (IN, OUT, OUT, OUT, OUT, OUT)),
    # x = nx - 1 starts a wave of its own, the other face its neighbour's; smallest open axis
    "d3q19_seam": (19, 65, 3, 9, (OUT, OUT, OUT, IN, PER, PER)),
    "d2q9": (9, 129, 5, 1, (IN, OUT, OUT, OUT, PER, PER)),
}


@pytest.mark.parametrize("box", sorted(BOXES))
@pytest.mark.parametrize("form", ["fp64", "fp32", "fp16"])
def test_outlet_faces_in_every_form(box, form):
    import torch
    q, nx, ny, nz, faces = BOXES[box]
    lat = W.LatticeSpec(q=q, nx=nx, ny=ny, nz=nz, tau=0.7, force=(1e-6, 0, 0), faces=faces,
                        face_u=((0.02, 0.001, 0.0),) * 6)
    _print_case(test="outlet forms", box=box, form=form)
    G, H = gpu_lattice(lat, None, form), gpu_lattice(lat, None, "fp64")
    G.set_f(torch.from_numpy(W.random_state(lat, 5, amp=1e-2)).cuda())
    G.rasterize(None)
    H.rasterize(None)
    w = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4 if q == 9 else
                 [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12).reshape(-1, 1, 1, 1)
    for step in range(3):  # both parities
        f0 = G.get_f()
        H.set_f(f0)
        H.step(1)
        G.step(1)
        ref, got = H.get_f().cpu().numpy(), G.get_f().cpu().numpy()
        size = max(np.abs(ref - w).max(), np.abs(f0.cpu().numpy() - w).max())
        tol = {"fp64": 1e-14, "fp32": 64 * 2.0 ** -24 * size,
               "fp16": (64 * 2.0 ** -24 + 2.0 ** -11) * size}[form]
        err = np.abs(got - ref).max()
        print(f"step {step}: err {err:.2e} tol {tol:.2e}", flush=True)
        assert err <= tol
