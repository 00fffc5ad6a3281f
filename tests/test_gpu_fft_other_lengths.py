"""The FFT line lengths that test_gpu_fft_lengths.py leaves out: the other
lengths with a kernel of their own (sides 8 to 500) and six of the nine sides up
to 512 that have none (162, 216, 270, 324, 432, 450; 250, 360 and 486 are
there), on each axis of a 3D grid, in 2D grids, whose first inverse pass is the
Hermitian one along axis 1, and in batches whose members' lengths have kernels
of their own or not: u and E against the oracle, a batch's members also against
their own plans, bit for bit.  The plans are one (float32) or two digits finer
than the tolerance, so that the transforms decide on a white-noise density."""
import numpy as np
import pytest

import oracle
import workloads as wl
from gpu_util import make_plan, rel_l2, say

pytestmark = pytest.mark.gpu
import torch  # noqa: E402

OWN = [8, 20, 30, 36, 50, 54, 100, 108, 150, 300, 480, 500]
OTHER = [162, 216, 270, 324, 432, 450]
TOL = {"fp64": 1e-10, "mixed": 1e-5}
PLAN = {"fp64": 1e-12, "mixed": 1e-6}


def _problem(n, prec):
    box = tuple(0.5 * v for v in n)
    if len(n) == 3:
        return wl.Problem("len", 3, n, box, wl.DIPOLE_3D, 6, 4, 8, axis=(0.48, 0.6, 0.64), eps=PLAN[prec],
                          precision=wl.FP64 if prec == "fp64" else wl.MIXED)
    return wl.Problem("len", 2, n, box, wl.COULOMB_2D, 12, 1, 16, eps=PLAN[prec],
                      precision=wl.FP64 if prec == "fp64" else wl.MIXED)


def _density(n, prec, seed):
    return np.random.default_rng(seed).uniform(0.0, 1.0, n).astype(np.float64 if prec == "fp64" else np.float32)


def _check(p, rho, u, E, tol, *what):
    r = rho.astype(np.float64)
    ref = oracle.evaluate(p, r)
    e = rel_l2(u.cpu().numpy(), ref.u)
    H = np.prod([b / m for b, m in zip(p.box, p.n)])
    ee = abs(E.item() - ref.energy_physical) / (0.5 * H * float(np.linalg.norm(r) * np.linalg.norm(ref.u)))
    say("length", p.n, *what, "%.2e %.2e" % (e, ee))
    assert e < tol and ee < tol


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("side", OWN + OTHER)
def test_length_3d(side, axis, prec):
    n = [18, 10, 12]
    n[axis] = side
    p = _problem(tuple(n), prec)
    rho = _density(n, prec, side * 8 + axis)
    plan = make_plan(p)
    u, E = plan.potential(torch.tensor(rho, device="cuda"))
    _check(p, rho, u, E, TOL[prec], prec)
    plan.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("side", [8, 36, 50, 108, 128, 300, 480, 500, 512, 162, 250, 432, 486])
def test_length_2d(side, axis, prec):
    n = [30, 30]
    n[axis] = side
    p = _problem(tuple(n), prec)
    rho = _density(n, prec, side * 8 + axis)
    plan = make_plan(p)
    u, E = plan.potential(torch.tensor(rho, device="cuda"))
    _check(p, rho, u, E, TOL[prec], prec)
    plan.close()


@pytest.mark.parametrize("nstreams", [1, 3])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("grids", [[(16, 12, 162), (216, 12, 10), (20, 250, 12), (24, 20, 16), (30, 50, 54)],
                                   [(324, 40), (36, 432), (486, 30), (32, 48), (100, 108)]])
def test_batch_of_lengths(grids, prec, nstreams):
    import paper_1311_4120_amd as jgb
    probs = [_problem(n, prec) for n in grids]
    kws = [dict(n=p.n, box=p.box, kernel="dipole3d" if p.dim == 3 else "coulomb2d",
                nodes=(p.n_r, p.n_theta, p.n_phi) if p.dim == 3 else (p.n_r, p.n_phi), eps=p.eps, precision=prec,
                axis=p.axis) for p in probs]
    rhos = [_density(p.n, prec, 7 + i) for i, p in enumerate(probs)]
    b = jgb.Batch(kws, nstreams=nstreams)
    dev = [torch.tensor(r, device="cuda") for r in rhos]
    u, E = b.bind(dev)
    for rep in range(2):
        b.run()
        torch.cuda.synchronize()
        for i, p in enumerate(probs):
            ue, Ee = b.plans[i].potential(dev[i])
            torch.cuda.synchronize()
            assert torch.equal(u[i], ue) and E[i].item() == Ee.item(), (rep, p.n)
    for i, p in enumerate(probs):
        _check(p, rhos[i], u[i], E[i], TOL[prec], prec, "batch")
    b.close()
