"""Every form of the grid transfers gives the same grids: restrictions in
tiles and by groups of lanes, the last one in its own launch (per-stage
timing) and in the stencils'; prolongations of the small levels in one launch,
by groups of lanes, and one thread per coarse point beyond 4096 of them.  q of
every level and E of every level against the oracle."""
import numpy as np
import pytest

from oracle import mls as M
from paper_1308_4005_amd import workloads as W

from gpu_common import rel_err, say

pytestmark = pytest.mark.gpu

BOX, LEVELS = (48.0, 46.0, 47.0), 4   # 48^3, 24^3, 12^3 and 6^3 points


@pytest.fixture(scope="module", params=[4, 6])
def system(request):
    w = W.fill_box(1500, BOX, seed=31)
    w.c6 = np.random.default_rng(32).uniform(1.0, 9.0, w.n)
    return request.param, w, M.mls(w.pos, w.c6, w.box, 2.5, 1.0, request.param, LEVELS)


@pytest.mark.parametrize("timing", [False, True], ids=["joint", "separate"])
@pytest.mark.parametrize("prolong", [None, "0", "9999999"])
@pytest.mark.parametrize("restrict", [None, "0", "9999999"])
def test_forms_agree(monkeypatch, system, restrict, prolong, timing):
    import torch
    from paper_1308_4005_amd import Plan
    order, w, ref = system
    for name, v in (("MLS_SPLIT_RESTRICT", restrict), ("MLS_SPLIT_PROLONG", prolong)):
        monkeypatch.setenv(name, v) if v else monkeypatch.delenv(name, False)
    plan = Plan(w.box, 2.5, 1.0, order, LEVELS, n_max=w.n)
    t = lambda x: torch.tensor(x, dtype=torch.float64, device="cuda")
    plan.set_timing(timing)
    plan.evaluate(t(w.pos), t(w.c6))
    worst = 0.0
    for k in range(1, LEVELS + 1):
        for name in ("q", "E"):
            worst = max(worst, rel_err(plan.copy_stage(name, k).cpu().numpy(), ref[name][k - 1]))
    say(f"[transfer forms] p={order} {restrict} {prolong} {timing}: {worst:.1e}")
    assert worst < 1e-12
    plan.close()
