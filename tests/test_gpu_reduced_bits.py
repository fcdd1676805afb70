"""The reduced forms' arithmetic, to the bit.  FP32 arithmetic is the same
operations in the same order on every run, so the populations after a few
steps are numbers that do not change: their CRC-32 is recorded in
tests/golden/reduced_populations.txt from the collision that multiplies every
direction's own sum by its split weight.  Sums formed once per cell and shared
by the directions pass every tolerance of the other tests and yet are further
from FP64 (an open box with a sphere: velocities 6 % in the geometric mean
over 16 placements, single torques twice).  No tolerance: equality."""
import os
import zlib

import numpy as np
import pytest

import workloads as W
from helpers import WALLS_Y, _particles, _print_case, gpu_lattice

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden",
                      "reduced_populations.txt")
PER, BB, MW, IN, OUT = W.PERIODIC, W.BOUNCE_BACK, W.MOVING_WALL, W.INLET_EQ, W.OUTLET_EQ
OPEN = (IN,) + (OUT,) * 5
WALLS_X = (BB, MW) + (PER,) * 4
FU = ((0.02, 0.001, 0.0), (0.0, 0.01, 0.0)) + ((0.0, 0.0, 0.0),) * 4
# q, nx, ny, nz, faces, body force, weighting
CASES = {
    "2d_periodic": (9, 128, 40, 1, (PER,) * 6, 0.0, "modified"),
    "2d_forced_walls": (9, 100, 41, 1, WALLS_Y, 2e-5, "modified"),
    "3d_periodic": (19, 64, 22, 20, (PER,) * 6, 0.0, "modified"),
    "3d_forced": (19, 64, 22, 20, (PER,) * 6, 2e-5, "modified"),
    "3d_short_rows": (19, 37, 22, 20, (PER,) * 6, 0.0, "modified"),
    "3d_walls": (19, 64, 22, 20, WALLS_X, 0.0, "modified"),
    "3d_forced_walls": (19, 70, 22, 20, WALLS_X, 2e-5, "modified"),
    "3d_open": (19, 70, 40, 20, OPEN, 0.0, "modified"),
    # flat waves with x = 0 in the last lane (65 y, 67 y = 63 mod 64) and x = nx - 1
    # in the first; x = 64 alone in its segment
    "3d_open_65": (19, 65, 70, 20, OPEN, 0.0, "modified"),
    "3d_out_65": (19, 65, 70, 20, (OUT, OUT, OUT, IN, PER, PER), 0.0, "modified"),
    "3d_out_67": (19, 67, 70, 20, (OUT, OUT, OUT, IN, PER, PER), 1e-5, "modified"),
    "2d_out_67": (9, 67, 70, 1, (OUT, OUT, OUT, IN, PER, PER), 1e-5, "modified"),
    "3d_original": (19, 64, 22, 20, (PER,) * 6, 0.0, "original"),
}


def crc(name, form):
    import torch
    import paper_1901_09745_amd.psclbm as P
    q, nx, ny, nz, faces, fx, weighting = CASES[name]
    lat = W.LatticeSpec(q=q, nx=nx, ny=ny, nz=nz, tau=0.65, force=(fx, 0.0, 0.0), faces=faces,
                        face_u=FU)
    p = _particles(lat, 6, 3.0, 4.5, seed=11, overlap=True)
    G = gpu_lattice(lat, p, form, weighting=weighting)
    G.set_f(torch.from_numpy(W.random_state(lat, 7, amp=1e-2)).cuda())
    G.rasterize(P.DeviceParticles.from_host(p))
    G.step(5)
    f = G.get_f()
    G.sync()
    return zlib.crc32(np.ascontiguousarray(f.cpu().numpy()).tobytes())


@pytest.mark.parametrize("form", ["fp32", "fp16"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_reduced_populations(name, form):
    _print_case(test="reduced populations", name=name, form=form)
    with open(GOLDEN) as f:
        want = {(a, b): int(c, 16) for a, b, c in (ln.split() for ln in f if ln[0] != "#")}
    assert crc(name, form) == want[name, form]
