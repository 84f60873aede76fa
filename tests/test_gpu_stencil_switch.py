"""Mixed plans that leave the FP32 tiles for the FP64 slab kernel
(MLS_STENCIL_KERNEL=0): every plane of every level's potential is written,
also where the FP32 tiles would have another depth (windows up to 6, extents
that are no multiple of either), and equals the default plan's within the
mixed bound on potentials, 1e-5 of the largest.  The plan under test comes
first, with charges of its own, so that no plane can hold the values of another
plan whose memory it was given."""
import numpy as np
import pytest

from paper_1308_4005_amd import workloads as W

from gpu_common import rel_err, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mixing", ["geometric", "lorentz-berthelot"])
@pytest.mark.parametrize("a,h,order,R", [(2.0, 1.0, 4, 4), (3.0, 1.0, 6, 6), (3.2, 0.8, 4, 8)])
def test_slab_stencil_of_a_mixed_plan(a, h, order, R, mixing, monkeypatch):
    import torch
    from paper_1308_4005_amd import Plan
    box = np.array([17.0, 18.0, 24.0])
    w = W.fill_box(3000, box, seed=11)
    rng = np.random.default_rng(R + (100 if mixing == "geometric" else 200))
    t = lambda x: torch.tensor(x, dtype=torch.float64, device="cuda")
    pos, sig = t(w.pos), t(rng.choice([0.9, 1.1], w.n))
    c6 = t(rng.uniform(1.0, 9.0, w.n))
    out = []
    for kernel in ("0", "1"):
        monkeypatch.setenv("MLS_STENCIL_KERNEL", kernel)
        plan = Plan(box, a, h, order, 2, n_max=w.n, precision="mixed", mixing=mixing)
        say(f"  grid {plan.info['grid']}")
        r = plan.evaluate(pos, c6) if mixing == "geometric" else plan.evaluate_lb(pos, c6, sig)
        e = [plan.copy_stage("e", k).cpu().numpy() for k in (1, 2)] if mixing == "geometric" else []
        out.append((e, r.energy.item(), r.forces.cpu().numpy()))
        plan.close()
    (e0, E0, F0), (e1, E1, F1) = out
    for x0, x1 in zip(e0, e1):
        say(f"[stencil switch] R={R} {mixing}: e rel={rel_err(x0, x1):.2e}")
        assert rel_err(x0, x1) < 1e-5
    assert abs(E0 - E1) < 1e-6 * abs(E1)
    assert rel_err(F0, F1) < 1e-5
