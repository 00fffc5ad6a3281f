"""The form and chunk of a tuned mixed-precision plan decide the last digits of
E, so they follow from what the plan counts and not from a timing
(csrc/formcost.h).  Each node set here gave the form and chunk below in plans
that timed them on the device, twice, every other one at least 3% slower; the
256^3 set stands for the two longest ring chunks, which cost the same there."""
import pytest

pytestmark = pytest.mark.gpu
import torch  # noqa: E402, F401

# grid, nodes, eps ("gauss": the Gaussian's 12 taps), Algorithm 2, tiles, gather
# chunk (negative: rings)
SETS = [
    ((16, 16, 16), (20, 10, 20), 1e-5, False, True, 256),
    ((24, 24, 24), (31, 15, 30), 1e-6, False, True, 256),
    ((32, 32, 32), (41, 20, 40), 1e-5, False, True, 256),
    ((40, 40, 40), (24, 12, 24), 1e-5, False, False, 256),
    ((40, 40, 40), (40, 20, 40), 1e-4, False, False, 256),
    ((48, 48, 48), (28, 14, 28), 1e-6, False, False, 256),
    ((64, 64, 64), (25, 12, 24), 1e-4, False, False, 256),
    ((64, 64, 64), (64, 32, 64), 1e-5, False, False, 512),
    ((64, 64, 64), (83, 41, 82), 1e-5, False, False, -2048),
    ((90, 60, 108), (27, 13, 26), 1e-5, False, False, 256),
    ((90, 60, 108), (108, 54, 108), 1e-5, False, False, -4096),
    ((90, 60, 108), (140, 70, 140), 1e-4, False, False, -4096),
    ((128, 64, 32), (102, 51, 102), 1e-4, False, False, 1024),
    ((96, 96, 96), (24, 12, 24), 1e-6, False, False, 256),
    ((96, 96, 96), (124, 62, 124), 1e-5, False, False, -4096),
    ((128, 128, 128), (32, 16, 32), 1e-4, False, True, 256),
    ((128, 128, 128), (76, 38, 76), 1e-6, False, False, 1024),
    ((128, 128, 128), (102, 51, 102), 1e-5, False, True, -4096),
    ((128, 128, 128), (128, 64, 128), 1e-5, False, True, -4096),
    ((160, 144, 160), (160, 80, 160), 1e-5, False, True, -8192),
    ((128, 128, 128), (20, 16, 32), 1e-6, True, True, 256),
    ((160, 144, 160), (28, 20, 40), 1e-4, True, True, 256),
    ((64, 64, 64), (40, 32, 64), 1e-4, True, False, 512),
    ((128, 128, 128), (40, 32, 64), 1e-6, True, False, -1024),
    ((256, 256, 256), (256, 128, 256), 1e-5, False, True, -8192),
    ((32, 32, 32), (32, 16, 32), "gauss", False, True, 256),
    ((48, 48, 48), (33, 16, 32), "gauss", False, False, 256),
    ((64, 64, 64), (64, 32, 64), "gauss", False, False, -2048),
    ((96, 96, 96), (96, 48, 96), "gauss", False, True, -4096),
    ((90, 60, 108), (108, 54, 108), "gauss", False, True, -4096),
    ((128, 128, 128), (40, 32, 64), "gauss", True, False, -1024),
    ((64, 64, 64), (64, 32, 64), 1e-2, False, False, 512),
    ((96, 96, 96), (96, 48, 96), 1e-2, False, False, 1024),
    ((160, 144, 160), (208, 104, 208), 1e-2, False, True, -8192),
]


@pytest.mark.parametrize("n,nodes,eps,split,tiles,chunk", SETS)
def test_form(n, nodes, eps, split, tiles, chunk, monkeypatch):
    import paper_1311_4120_amd as jgb
    monkeypatch.delenv("JGB_AUTOTUNE_CACHE", raising=False)
    gauss = eps == "gauss"
    plan = jgb.Plan(n, tuple(0.15 * v for v in n), "dipole3d", nodes, eps=1e-5 if gauss else eps, precision="mixed",
                    gaussian_kernel=gauss, axis=(0.48, 0.6, 0.64), theta_rule="costheta" if split or n[0] == 256 else "theta", split=split,
                    autotune=True)
    got = plan.info["interp_chunk"] == 0, plan.info["spread_chunk"]
    plan.close()
    print("mixed form", n, nodes, eps, split, got, flush=True)
    assert got == (tiles, chunk)


@pytest.mark.parametrize("n,nodes,tiles", [((64, 64, 64), (64, 32, 64), False), ((96, 96, 96), (76, 38, 76), False),
                                           ((32, 32, 32), (32, 16, 32), True)])
def test_no_tables_for_a_refused_form(n, nodes, tiles, monkeypatch):
    """Tuning a mixed plan that keeps the staged interpolation costs no device
    memory: the plan holds what the same plan untuned does (with the ring
    tables, which the choice of the spreading needs)."""
    import paper_1311_4120_amd as jgb
    monkeypatch.delenv("JGB_AUTOTUNE_CACHE", raising=False)
    kw = dict(eps=1e-5, precision="mixed", axis=(0.48, 0.6, 0.64), spread_rings=True)
    box = tuple(0.15 * v for v in n)
    plain, tuned = jgb.Plan(n, box, "dipole3d", nodes, **kw), jgb.Plan(n, box, "dipole3d", nodes, autotune=True, **kw)
    got = [p.info["workspace_bytes"] for p in (plain, tuned)]
    form = tuned.info["interp_chunk"] == 0
    plain.close()
    tuned.close()
    print("tables", n, nodes, got, flush=True)
    assert form == tiles and (got[1] > got[0] if tiles else got[1] == got[0])
