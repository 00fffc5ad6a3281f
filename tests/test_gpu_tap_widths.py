"""The interpolation by tiles and the spreading by rings at every kernel width
their record copies are compiled for, against the default forms, on grids whose
sides end inside a tile and, for the interpolation, on one so small that
footprints wrap around a tile.  Both forms add the same terms in the same
precision: at most w^3 per node or grid point, in partial sums of about 3 w
roundings, so they agree to a few ulps of the largest partial sums (1e-13 in
float64, 2e-6 in float32)."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import MODES, make_plan, rel_l2, say

pytestmark = pytest.mark.gpu
import torch  # noqa: E402

EPS = {"fp64": ["1e-%d" % k for k in range(2, 14)], "mixed": ["1e-%d" % k for k in range(2, 7)]}


@pytest.mark.parametrize("n,mode", [((30, 18, 50), "tiles+rings"), ((40, 18, 54), "tiles+rings"), ((8, 10, 10), "tiles")])
@pytest.mark.parametrize("prec,eps", [(p, e) for p in EPS for e in EPS[p]])
def test_forms_agree(prec, eps, n, mode):
    eps = float(eps)
    box = tuple(0.5 * v for v in n)
    p = wl.Problem("tap", 3, n, box, wl.DIPOLE_3D, 20, 12, 24, axis=(0.48, 0.6, 0.64))
    dt = torch.float64 if prec == "fp64" else torch.float32
    rho = torch.tensor(np.random.default_rng(3).uniform(0.0, 1.0, n), dtype=dt, device="cuda")
    forms, plain = make_plan(p, eps=eps, precision=prec, **MODES[mode]), make_plan(p, eps=eps, precision=prec)
    try:
        assert forms.info["interp_chunk"] == 0
        a, b = forms.transform(rho), plain.transform(rho)
        ua, Ea = forms.potential(rho)
        ub, Eb = plain.potential(rho)
        et, eu = rel_l2(a.cpu().numpy(), b.cpu().numpy()), rel_l2(ua.cpu().numpy(), ub.cpu().numpy())
        say("tap", prec, eps, n, mode, "%.2e %.2e" % (et, eu))
        tol = 1e-13 if prec == "fp64" else 2e-6
        assert et < tol and eu < tol
    finally:
        forms.close()
        plain.close()
