"""Neighbour reuse in mixed precision: on a step that does not bin again the
FP32 stencil tiles still hold the charges minus their own mean.  e^1 of such a
step against a plan that bins at the same positions, with the tiles adding up
the charges' sum themselves (up to 65520 atoms) and with the sum's own kernel.
Both plans round the same differences to FP32 and add them with the same
weights in the same order, so they agree to a few FP32 roundings (16); a mean
that is off by a factor loses that factor's bits (here 10^3)."""
import numpy as np
import pytest

from paper_1308_4005_amd import workloads as W

from gpu_common import rel_err, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,box", [(2000, (13.0, 14.0, 15.0)), (66000, (43.0, 44.0, 45.0))])
def test_charge_mean_of_a_reused_binning(n, box):
    import torch
    from paper_1308_4005_amd import Plan
    w = W.fill_box(n, np.array(box), seed=13)
    rng = np.random.default_rng(14)
    t = lambda x: torch.tensor(x, dtype=torch.float64, device="cuda")
    c6, c12, im = t(rng.uniform(1.0e4, 2.0e4, n)), t(np.full(n, 4.0)), t(np.full(n, 1e-12))
    plans = [Plan(w.box, 3.0, 1.0, 4, 2, n_max=n, precision="mixed", skin=0.2) for _ in range(2)]
    x = t(w.pos)
    plans[0].md_run(x, t(rng.uniform(-1.0, 1.0, (n, 3))), c6, c12, im, dt=1e-3, nsteps=2)
    assert (x - t(w.pos)).abs().max().item() < 0.05   # no atom near skin / 2
    plans[1].evaluate(x, c6)
    e = [p.copy_stage("e", 1).cpu().numpy() for p in plans]
    say(f"[md reuse] n={n}: e rel={rel_err(e[0], e[1]):.2e}")
    assert rel_err(e[0], e[1]) < 16 * 2.0 ** -23
    for p in plans:
        p.close()
