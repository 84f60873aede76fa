"""FP64 level stencils that stream their tile through LDS in slabs of z planes
(windows 7..12, both tile depths of the plan's rule), against the tap-by-tap
oracle on the GPU plan's own level-1 and level-2 charges: grids smaller than
the halo, ragged against the 8 x 8 x 8 and 8 x 8 x 16 tiles, and large enough
for the deep tiles."""
import numpy as np
import pytest

from oracle import mls as M

pytestmark = pytest.mark.gpu

# box, a, explicit finest grid, window
CASES = [
    ((7.0, 8.75, 10.5), 3.6, (8, 10, 12), 8),              # narrower than the window
    ((17.0, 18.0, 37.0), 4.0, (18, 20, 42), 9),            # R = 9, ragged in every dimension
    ((16.0, 16.0, 24.0), 3.6, (22, 24, 34), 10),
    ((12.0, 14.0, 20.0), 3.4, (20, 24, 36), 12),
    ((40.0, 38.0, 60.0), 3.5, (72, 68, 108), 12),          # 292 deep tiles: depth 16
    ((100.0, 96.0, 120.0), 3.9, (100, 98, 122), 7),        # more than 1024 deep tiles: depth 16
]


@pytest.mark.parametrize("box,a,grid,R", CASES, ids=[f"R{c[3]}_{'x'.join(map(str, c[2]))}" for c in CASES])
def test_slab_stencil_equals_taps(box, a, grid, R):
    import torch
    from paper_1308_4005_amd import Plan
    rng = np.random.default_rng(R)
    n = 400
    plan = Plan(box, a, order=4, levels=2, grid=grid, n_max=n)
    assert plan.info["stencil_path"] == ("tile_f64" if R <= 8 else "stream_f64")
    pos = torch.tensor(rng.uniform(0, 1, (n, 3)) * np.array(box), device="cuda")
    plan.evaluate(pos, torch.tensor(rng.uniform(1.0, 4.0, n), device="cuda"))
    q, e = plan.copy_stage("q", 1).cpu().numpy(), plan.copy_stage("e", 1).cpu().numpy()
    h1 = np.array(box) / np.array(grid)
    off, w = M.stencil_taps(h1, a)
    assert np.abs(off).max() == R
    # periodic convolution of the taps with the plan's charges
    k = np.zeros(q.shape)
    np.add.at(k, tuple(np.mod(off[:, d], q.shape[2 - d]) for d in (2, 1, 0)), w)
    ref = np.fft.irfftn(np.fft.rfftn(q) * np.fft.rfftn(k), s=q.shape, axes=(0, 1, 2))
    # a few thousand FP64 terms per point
    assert np.max(np.abs(e - ref)) <= 1e-12 * np.max(np.abs(ref))
    plan.close()
