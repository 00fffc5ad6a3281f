"""Every line length with an FFT kernel of its own, and neighbours without one,
on each axis of a 3D grid (the other sides leave partly filled blocks), by both
algorithms: u and E against the oracle's direct sums.  The density is white
noise, whose corner frequencies meet the spreading kernel's largest errors; in
float64 the plan is two digits finer than the tolerance, so that the transforms
decide."""
import numpy as np
import pytest

import oracle
import workloads as wl
from gpu_util import make_plan, rel_l2, say
from oracle import split

pytestmark = pytest.mark.gpu
import torch  # noqa: E402

SIDES = [16, 24, 32, 40, 48, 64, 72, 80, 96, 120, 128, 144, 160, 192, 200, 240, 256, 288, 320, 384, 400, 512,
         18, 60, 90, 180, 250, 360, 486]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("alg", [1, 2])
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("side", SIDES)
def test_length(side, axis, alg, prec):
    n = [18, 10, 12]
    n[axis] = side
    eps = 1e-10 if prec == "fp64" else 1e-5
    box = tuple(0.5 * v for v in n)
    p = wl.Problem("len", 3, tuple(n), box, wl.DIPOLE_3D, 6, 4, 8, axis=(0.48, 0.6, 0.64), eps=eps,
                   precision=wl.FP64 if prec == "fp64" else wl.MIXED)
    rng = np.random.default_rng(side * 8 + axis)
    rho = rng.uniform(0.0, 1.0, n).astype(np.float64 if prec == "fp64" else np.float32)
    plan = make_plan(p, split=(alg == 2), eps=1e-12 if prec == "fp64" else eps)
    u, E = plan.potential(torch.tensor(rho, device="cuda"))
    r = rho.astype(np.float64)
    if alg == 1:
        ref = oracle.evaluate(p, r)
        ur, Er = ref.u, ref.energy_physical
    else:
        ur, _, _, Er = split.potential_split(p, r)
    e = rel_l2(u.cpu().numpy(), ur)
    H = np.prod([b / m for b, m in zip(box, n)])
    ee = abs(E.item() - Er) / (0.5 * H * float(np.linalg.norm(r) * np.linalg.norm(ur)))
    say("length", side, axis, alg, prec, "%.2e %.2e" % (e, ee))
    assert e < eps and ee < eps
    plan.close()
