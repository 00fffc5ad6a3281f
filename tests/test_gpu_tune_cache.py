"""The tuning file: a plan with a forced form must not leave that form to plans
without one.  In mixed precision a plain plan's choices are the same without a
file, after a forced plan of the same shape and after another plain plan; a
forced plan still takes a plain plan's entry where it fits."""
import json

import pytest

pytestmark = pytest.mark.gpu
import torch  # noqa: E402, F401


def _plan(prec="mixed", **kw):
    import paper_1311_4120_amd as jgb
    plan = jgb.Plan((32, 32, 32), (8.0, 8.0, 8.0), "dipole3d", (32, 16, 32), eps=1e-5, precision=prec,
                    axis=(0.48, 0.6, 0.64), autotune=True, **kw)
    got = plan.info["interp_chunk"], plan.info["spread_chunk"]
    plan.close()
    return got


@pytest.mark.parametrize("forced", [{"interp_tiles": True}, {"spread_rings": True},
                                    {"interp_tiles": True, "spread_rings": True}])
def test_forced_form_stays_with_its_plans(forced, tmp_path, monkeypatch):
    monkeypatch.delenv("JGB_AUTOTUNE_CACHE", raising=False)
    plain = _plan()
    cache = tmp_path / "tune.json"
    monkeypatch.setenv("JGB_AUTOTUNE_CACHE", str(cache))
    first = _plan(**forced)
    assert first[0] == 0 or "interp_tiles" not in forced
    assert first[1] < 0 or "spread_rings" not in forced
    assert _plan() == plain
    assert _plan() == plain and _plan(**forced) == first
    assert len(json.loads(cache.read_text())) == 2


def test_forced_plan_reads_a_plain_entry(tmp_path, monkeypatch):
    cache = tmp_path / "tune.json"
    monkeypatch.setenv("JGB_AUTOTUNE_CACHE", str(cache))
    plain = _plan("fp64")
    assert _plan("fp64", interp_tiles=True) == (0, plain[1])
    assert len(json.loads(cache.read_text())) == 1
