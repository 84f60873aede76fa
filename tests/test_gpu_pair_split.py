"""Pair kernels that deal the rows of 64 targets to several waves, against the
kernels where one wave scans all rows (a plan created with a persistent grid
option keeps those): the same pairs, and in mixed precision the same FP32
sums, so the local potentials and forces agree to FP64 rounding at every edge
of the rule (idle lanes, one and several blocks, 8 / 4 / 2 / 1 waves) and for
a box with more neighbours than the mixed kernel's lists hold."""
import numpy as np
import pytest

from paper_1308_4005_amd import workloads as W

pytestmark = pytest.mark.gpu

# sums of a few hundred FP64 terms in another order
TOL = 1e-13


def _jittered(n, side, cells, seed):
    """n of cells^3 lattice sites, each atom moved by up to a tenth of the spacing."""
    rng = np.random.default_rng(seed)
    s = side / cells
    sites = rng.permutation(cells ** 3)[:n]
    x = np.stack([sites % cells, sites // cells % cells, sites // cells ** 2], 1)
    return (x + 0.5 + rng.uniform(-0.1, 0.1, (n, 3))) * s


def _plan(monkeypatch, one_wave, box, a, precision, n, mixing):
    from paper_1308_4005_amd import Plan
    # more persistent blocks than groups: the ordinary launch of the one-wave kernels
    monkeypatch.setenv("MLS_PAIR_WAVES_CU", "64") if one_wave else monkeypatch.delenv("MLS_PAIR_WAVES_CU", False)
    return Plan(box, a, 1.0, 4, 0, precision=precision, n_max=n, mixing=mixing)


CASES = [
    ("one", 1, 9.0, 3.0), ("wave", 64, 9.0, 3.0), ("wave+1", 65, 9.0, 3.0), ("liquid", 3000, 15.5, 3.0),
    ("gas", 700, 40.0, 2.5), ("full", 2197, 10.4, 4.15 / 2), ("crowded", 9000, 16.8, 3.3),
    ("8 waves", 32768, 36.0, 3.0), ("4 waves", 32769, 36.0, 3.0), ("2 waves", 65537, 45.0, 3.0),
    ("1 wave", 131073, 56.0, 3.0),
]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_split_rows_equal_one_wave(monkeypatch, case, precision):
    import torch
    _, n, side, a = case
    cells = max(2, int(np.ceil(n ** (1 / 3) - 1e-9)))
    t = lambda x: torch.tensor(x, dtype=torch.float64, device="cuda")
    pos = t(_jittered(n, side, cells, n))
    rng = np.random.default_rng(n + 1)
    c6, c12 = t(rng.uniform(0.0, 4.0, n)), t(rng.uniform(0.0, 4.0, n))
    eps, sig = t(rng.uniform(0.5, 1.0, n)), t(rng.uniform(0.9, 1.3, n))
    got = []
    for one_wave in (True, False):
        out = []
        for mixing in ("geometric", "lb") if n < 5000 else ("geometric",):
            p = _plan(monkeypatch, one_wave, (side,) * 3, a, precision, n, mixing)
            # per-stage timing runs the local part alone, as small evaluations do
            p.set_timing(True)
            if mixing == "geometric":
                r = p.evaluate_md(pos, c6, c12)
                out += [r.energy, r.forces]
                p.evaluate(pos, c6)
            else:
                p.evaluate_lb(pos, eps, sig)
            out += [p.copy_stage("e0", n=n), p.copy_stage("floc", n=n)]
            torch.cuda.synchronize()
            assert p.status() == 0
            p.close()
        got.append(out)
    for x, y in zip(*got):
        assert torch.isfinite(x).all()
        assert (x - y).abs().max().item() <= TOL * max(x.abs().max().item(), 1e-300)
