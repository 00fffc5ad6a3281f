"""Batches whose members differ in what the kernels are compiled for: members
of different accuracies share every launch but the staged interpolation's (one
per width), and every result equals the member's own evaluation bit for bit."""
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu
import torch  # noqa: E402


def _kw(n, eps, prec, nodes=(12, 8, 16)):
    return dict(n=n, box=tuple(0.5 * v for v in n), kernel="dipole3d" if len(n) == 3 else "coulomb2d",
                nodes=nodes if len(n) == 3 else (nodes[0], nodes[2]), eps=eps, precision=prec, axis=(0.48, 0.6, 0.64))


@pytest.mark.parametrize("n", [(32, 30, 36), (48, 40)])
def test_launches_of_mixed_accuracies(n):
    import paper_1311_4120_amd as jgb
    count = {}
    for epss in [(1e-6, 1e-6, 1e-6), (1e-10, 1e-10, 1e-10), (1e-6, 1e-10, 1e-13)]:
        b = jgb.Batch([_kw(n, e, "fp64") for e in epss], nstreams=1)
        rhos = [torch.rand(n, dtype=torch.float64, device="cuda") for _ in epss]
        u, E = b.bind(rhos)
        count[epss] = b.launches()
        b.run()
        torch.cuda.synchronize()
        for i in range(3):
            ue, Ee = b.plans[i].potential(rhos[i])
            torch.cuda.synchronize()
            assert torch.equal(u[i], ue) and E[i].item() == Ee.item(), (epss, i)
        b.close()
    say("launches", n, count)
    # (the larger of the two: at 1e-10 some tiles are split and summed by a launch of its own)
    low, high, mixed = count.values()
    assert mixed == max(low, high) + 2
