"""The level stencils' launch with the coarsest level and the charges' sum in
it: a coarsest grid beyond the 2048 points that its blocks stage in LDS,
against the oracle (1e-12), and mixed-precision atom counts on both sides of
the one up to which the tiles add the sum themselves (65520), against the FP64
plan within the precision's stated bounds."""
import numpy as np
import pytest

from oracle import mls as M
from paper_1308_4005_amd import workloads as W

from gpu_common import force_errors, gpu_eval, rel_err, say, stages

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("box,coarsest", [((24.0, 24.0, 24.0), (12, 12, 12)), ((28.0, 28.0, 28.0), (14, 14, 14))])
def test_coarsest_in_the_stencil_launch(box, coarsest):
    w = W.fill_box(int(0.1 * np.prod(box)), np.array(box), seed=7)
    w.c6 = np.random.default_rng(8).uniform(1.0, 9.0, w.n)
    ref = M.mls(w.pos, w.c6, w.box, 2.5, 1.0, 4, 2)
    plan, _ = gpu_eval(w.pos, w.c6, w.box, 2.5, 1.0, 4, 2)
    st = stages(plan, w.n)
    assert st["e"][1].shape == coarsest
    for k in (0, 1):
        de = rel_err(st["e"][k], ref["e"][k])
        say(f"[joint] {coarsest} level {k + 1}: e rel={de:.2e}")
        assert de < 1e-12
    plan.close()


@pytest.mark.parametrize("n", [65520, 65521])
def test_charge_sum_in_the_tiles(n):
    w = W.fill_box(n, np.array([43.0, 44.0, 45.0]), seed=9)
    w.c6 = np.random.default_rng(10).uniform(1.0, 9.0, n)
    plan, ref = gpu_eval(w.pos, w.c6, w.box, 3.0, 1.0, 4, 3)
    plan.close()
    plan, out = gpu_eval(w.pos, w.c6, w.box, 3.0, 1.0, 4, 3, precision="mixed")
    plan.close()
    dE = abs(out["energy"] - ref["energy"]) / abs(ref["energy"])
    say(f"[joint] n={n}: dE={dE:.2e}")
    assert dE < 1e-6
    assert np.max(np.abs(out["u"] - ref["u"])) < 1e-5 * np.max(np.abs(ref["u"]))
    assert force_errors(out["F"], ref["F"])[0] < 1e-5
