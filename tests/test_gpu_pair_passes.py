"""The mixed-precision pair kernel of eight waves where one pass over the 25
rows does not fit its lists: lattices with many filter steps, cutoffs with
more neighbours than a list holds (two, four and more passes, queue entries
carried between them), and rows beyond the lists themselves (taken in parts).  Against the kernel where one wave scans all rows, which adds the
same FP32 terms in the same groups: equal to FP64 rounding."""
import numpy as np
import pytest

from test_gpu_pair_split import TOL, _jittered, _plan

pytestmark = pytest.mark.gpu

# name, atoms, side of the box and of the filled part, cutoff
CASES = [("lattice", 500, 8.55, 8.55, 3.0), ("steps", 4000, 17.1, 17.1, 3.0), ("one or two", 3375, 16.2, 16.2, 4.4),
         ("two", 3001, 15.5, 15.5, 5.0), ("four", 4096, 17.3, 17.3, 6.0), ("eight", 6000, 16.1, 16.1, 6.2),
         ("row", 12000, 9.05, 9.05, 3.6), ("blob", 5000, 15.5, 1.45, 3.0)]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_passes_equal_one_wave(monkeypatch, case):
    import torch
    _, n, side, filled, a = case
    cells = int(np.ceil(n ** (1 / 3) - 1e-9))
    t = lambda x: torch.tensor(x, dtype=torch.float64, device="cuda")
    pos = t(_jittered(n, filled, cells, n))
    rng = np.random.default_rng(n + 1)
    c6, c12 = t(rng.uniform(0.0, 4.0, n)), t(rng.uniform(0.0, 4.0, n))
    eps, sig = t(rng.uniform(0.5, 1.0, n)), t(rng.uniform(0.9, 1.3, n))
    got = []
    for one_wave in (True, False):
        out = []
        for mixing in ("geometric", "lb"):
            p = _plan(monkeypatch, one_wave, (side,) * 3, a, "mixed", n, mixing)
            p.set_timing(True)   # the local part alone, whatever the size
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
        assert (x - y).abs().max().item() <= TOL * x.abs().max().item()
