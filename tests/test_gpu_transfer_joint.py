"""The grid transfers that share launches with other work: the last restriction
in the coarsest level's blocks (up to 585 coarsest points) and the small levels'
prolongations in LDS (levels of up to 4096 points), on both sides of each
limit and for both orders; every level's charges, stencil sums and potentials
against the FP64 oracle (1e-12)."""
import numpy as np
import pytest

from oracle import mls as M
from paper_1308_4005_amd import workloads as W

from gpu_common import gpu_eval, rel_err, say, stages

pytestmark = pytest.mark.gpu

# box (spacing 1) and levels
CASES = {
    "coarsest585": ((10.0, 18.0, 26.0), 2),
    "coarsest588": ((14.0, 14.0, 24.0), 2),
    "odd_l3": ((12.0, 20.0, 28.0), 3),
    "level4096": ((32.0, 32.0, 32.0), 3),
    "level4352": ((34.0, 32.0, 32.0), 2),
    "deep_l5": ((16.0, 32.0, 32.0), 5),
}


@pytest.mark.parametrize("order", [4, 6])
@pytest.mark.parametrize("name", list(CASES))
def test_joint_transfers_match_oracle(name, order):
    box, levels = CASES[name]
    w = W.fill_box(int(0.06 * np.prod(box)), np.array(box), seed=31)
    w.c6 = np.random.default_rng(32).uniform(1.0, 9.0, w.n)
    ref = M.mls(w.pos, w.c6, w.box, 2.5, 1.0, order, levels)
    plan, out = gpu_eval(w.pos, w.c6, w.box, 2.5, 1.0, order, levels)
    st = stages(plan, w.n)
    for k in range(levels):
        d = [rel_err(st[key][k], ref[key][k]) for key in ("q", "e", "E")]
        say(f"[joint transfers] {name} p{order} level {k + 1}: " + " ".join(f"{v:.1e}" for v in d))
        assert max(d) < 1e-12
    assert out["energy"] == pytest.approx(ref["energy"], rel=1e-10)
    plan.close()


@pytest.mark.parametrize("order", [4, 6])
@pytest.mark.parametrize("name", ["odd_l3", "level4352", "deep_l5"])
def test_tiled_restriction_matches_oracle(name, order, monkeypatch):
    """Every restriction in tiles of 8 x 8 x 4 coarse points: levels smaller than
    a tile, ragged last tiles, fine extents below the taps' reach (1e-12)."""
    monkeypatch.setenv("MLS_SPLIT_RESTRICT", "0")
    box, levels = CASES[name]
    w = W.fill_box(int(0.06 * np.prod(box)), np.array(box), seed=33)
    w.c6 = np.random.default_rng(34).uniform(1.0, 9.0, w.n)
    ref = M.mls(w.pos, w.c6, w.box, 2.5, 1.0, order, levels)
    plan, _ = gpu_eval(w.pos, w.c6, w.box, 2.5, 1.0, order, levels)
    # timed stages run the last restriction in its own launch
    plan.set_timing(True)
    import torch
    plan.evaluate(*(torch.tensor(x, dtype=torch.float64, device="cuda") for x in (w.pos, w.c6)))
    st = stages(plan, w.n)
    for k in range(levels):
        d = rel_err(st["q"][k], ref["q"][k])
        say(f"[tiled restriction] {name} p{order} level {k + 1}: q {d:.1e}")
        assert d < 1e-12
    plan.close()
