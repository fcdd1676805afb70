"""The FP16 form's state as read out: f = w rho0 + h w of each stored half h,
rounded once (rho0 = 1, so w rho0 is w itself).  The reference is the same
sum in rational arithmetic, rounded to FP64.  No tolerance: equality."""
from fractions import Fraction

import numpy as np
import pytest

import workloads as W
from helpers import _print_case, gpu_lattice

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q", [9, 19])
def test_fp16_populations_are_rounded_once(q):
    import torch
    lat = W.LatticeSpec(q=q, nx=17, ny=9, nz=1 if q == 9 else 4, tau=0.7)
    _print_case(test="fp16 state", q=q)
    w = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4 if q == 9 else
                 [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)
    f0 = W.random_state(lat, 3, amp=0.3).reshape(q, -1)
    G = gpu_lattice(lat, None, "fp16")
    G.set_f(torch.from_numpy(f0).cuda())
    got = G.get_f().cpu().numpy().reshape(q, -1)
    h = ((f0 - w[:, None]) / w[:, None]).astype(np.float32).astype(np.float16)
    for i in range(q):
        wi = Fraction(float(w[i]))
        want = np.array([float(wi + Fraction(float(v)) * wi) for v in h[i]])
        assert np.array_equal(got[i], want), i
