"""The binning's forms by size, each against the oracle's stable counting sort
bit for bit: one block for up to 4096 atoms in up to 2048 cells; histograms of
up to 8192 entries added up by their readers, larger ones scanned.  And the
sorted sqrt(C12) that the sort writes for molecular dynamics against the
counting sort's gather: the same permutation, so the same sums up to the order
of the anterpolation's FP64 atomics (1e-12)."""
import numpy as np
import pytest

from gpu_common import gpu_eval, say
from test_gpu_binning import A, H, P, _check, _uniform

pytestmark = pytest.mark.gpu

CASES = [
    # 12^3 cells; around the block's 64, 1024 and 4096 atoms
    *[(f"n{n}", n, (18.0, 18.0, 18.0), None) for n in (1, 65, 1025, 4095, 4096, 4097)],
    # 2048 cells, and 2176 in five buckets
    ("cells2048", 3000, (12.0, 24.0, 24.0), None),
    ("cells2176", 3000, (12.0, 24.0, 25.5), None),
    # every atom in one cell of the block
    ("one_cell", 4096, (18.0, 18.0, 18.0), (1.4, 1.4, 1.4)),
    # 128 buckets: 64 blocks of atoms and one more
    ("hist8192", 131072, (48.0, 48.0, 96.0), None),
    ("hist8320", 131073, (48.0, 48.0, 96.0), None),
]


@pytest.mark.parametrize("k", range(len(CASES)), ids=[c[0] for c in CASES])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_sort_by_size(k, precision):
    name, n, box, hi = CASES[k]
    w = _uniform(n, box, 20 + k, hi=hi)
    say(f"[bin small] {name} {precision}: n={n}")
    plan, _ = gpu_eval(w.pos, w.c6, w.box, A, H, P, 1, precision=precision)
    _check(w, plan)
    plan.close()


@pytest.mark.parametrize("n", [1, 4096, 4097])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_repulsion_from_the_sort(n, precision, monkeypatch):
    import torch
    from paper_1308_4005_amd import Plan
    w = _uniform(n, (18.0, 18.0, 18.0), 50)
    c12 = np.random.default_rng(51).uniform(0.5, 2.0, n)
    bad = c12.copy()
    bad[n - 1] = np.nan
    pos, c6, tc, tb = (torch.tensor(x, dtype=torch.float64, device="cuda") for x in (w.pos, w.c6, c12, bad))
    out = []
    for buckets in ("0", "1"):
        monkeypatch.setenv("MLS_BIN_BUCKETS", buckets)
        plan = Plan(w.box, A, H, P, 1, n_max=n, precision=precision)
        r = plan.evaluate_md(pos, c6, tc, rc=2.0)
        assert plan.status() == 0
        out.append((float(r.energy.cpu()[0]), r.forces.cpu().numpy()))
        plan.evaluate_md(pos, c6, tb, rc=2.0)
        assert plan.status() & 8
        plan.close()
    say(f"[bin small] repulsion {precision} n={n}: E={out[1][0]:.6e}")
    assert out[1][0] == pytest.approx(out[0][0], rel=1e-12)
    np.testing.assert_allclose(out[1][1], out[0][1], rtol=0, atol=1e-12 * np.max(np.abs(out[0][1])))
