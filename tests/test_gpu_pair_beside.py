"""The FP32 pair kernel as a grid of fewer blocks than groups of 64 targets,
each block walking several groups (large mixed plans beside the grid chain;
here forced at a small size): every group's sums are its own, so e_0 and the
local forces equal the one-group-per-block launch bit for bit."""
import numpy as np
import pytest

from paper_1308_4005_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mixing", ["geometric", "lorentz-berthelot"])
@pytest.mark.parametrize("n", [33000, 32768 + 16384 + 1])   # 516 and 769 groups over 256 blocks
def test_groups_shared_by_blocks(n, mixing, monkeypatch):
    import torch
    from paper_1308_4005_amd import Plan
    w = W.fill_box(n, np.array([37.0, 38.0, 39.0]), seed=3)
    rng = np.random.default_rng(4)
    t = lambda x: torch.tensor(x, dtype=torch.float64, device="cuda")
    pos, c6, sig = t(w.pos), t(rng.uniform(0.5, 4.0, n)), t(rng.uniform(0.8, 1.2, n))
    out = []
    for waves in ("64", "1"):   # per compute unit: more blocks than groups, and 256 blocks
        monkeypatch.setenv("MLS_PAIR_WAVES_CU", waves)
        plan = Plan(w.box, 3.0, 1.0, 4, 2, n_max=n, precision="mixed", mixing=mixing)
        if mixing == "geometric":
            plan.evaluate(pos, c6)
        else:
            plan.evaluate_lb(pos, c6, sig)
        out.append((plan.copy_stage("e0", n=n).cpu(), plan.copy_stage("floc", n=n).cpu()))
        plan.close()
    assert torch.isfinite(out[0][0]).all()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
