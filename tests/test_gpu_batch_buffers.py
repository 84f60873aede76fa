"""Batched evaluations that change the caller's arrays from call to call: other
inputs, fresh and reused outputs, outputs left out, another stream, and a
captured evaluation replayed between eager ones with other arrays.  Each call
against the same boxes evaluated once with arrays of its own."""
import numpy as np
import pytest

from paper_1308_4005_amd import workloads as W

pytestmark = pytest.mark.gpu

SIZES = [(300, (9.0, 9.0, 9.0)), (900, (12.0, 10.0, 14.0)), (0, (8.0, 8.0, 8.0)), (120, (5.0, 5.0, 8.0))]


def _inputs(seed, lb):
    import torch
    t = lambda x: torch.tensor(x, dtype=torch.float64, device="cuda")
    rng = np.random.default_rng(seed)
    pos = np.concatenate([W.fill_box(n, b, seed=100 * seed + k).pos for k, (n, b) in enumerate(SIZES) if n])
    n = len(pos)
    per = (t(rng.uniform(0.5, 1, n)), t(rng.choice([1.0, 1.2], n))) if lb else (t(rng.uniform(1, 9, n)),)
    return (t(pos),) + per


def _plan(lb):
    from paper_1308_4005_amd import BatchPlan
    return BatchPlan([b for _, b in SIZES], [n for n, _ in SIZES], 2.5, 1.0, 4, mixing="lb" if lb else "geometric")


def _run(bp, lb, x, **kw):
    return bp.evaluate_lb(*x, **kw) if lb else bp.evaluate(*x, dE_dc6=True, **kw)


def _same(r, ref):
    for k in ("energies", "forces", "dE_dc6"):
        a, b = getattr(r, k), getattr(ref, k)
        if a is not None:   # FP64 atomics: the last bits vary
            assert (a - b).abs().max() <= 1e-12 * b.abs().max()


@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("lb", [False, True], ids=["geometric", "lb"])
def test_changing_arrays(lb, graph):
    import torch
    sets = [_inputs(s, lb) for s in (1, 2, 3)]
    ref = [_run(_plan(lb), lb, x) for x in sets]
    bp = _plan(lb)
    bp.set_graph(graph)
    kept = [_run(bp, lb, sets[k % 3]) for k in range(5)]        # fresh outputs, all alive
    for k in (2, 0, 1, 1, 2):                                    # reused ones
        kept[k] = _run(bp, lb, sets[(k + 1) % 3], out=kept[k])
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        other = _run(bp, lb, sets[2])
    torch.cuda.current_stream().wait_stream(side)
    part = bp.evaluate_lb(*sets[0], forces=False) if lb else bp.evaluate(*sets[0], forces=False)
    assert part.forces is None
    torch.cuda.synchronize()
    for k in range(5):
        _same(kept[k], ref[(k + 1) % 3] if k < 3 else ref[k % 3])
    _same(other, ref[2])
    _same(part, ref[0])
    assert bp.status() == 0


@pytest.mark.parametrize("lb", [False, True], ids=["geometric", "lb"])
def test_captured_evaluation_between_eager_ones(lb):
    import torch
    sets = [_inputs(s, lb) for s in (1, 2)]
    ref = [_run(_plan(lb), lb, x) for x in sets]
    bp = _plan(lb)
    bp.set_graph(False)
    a, b = _run(bp, lb, sets[0]), _run(bp, lb, sets[1])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        _run(bp, lb, sets[0], out=a)
    for _ in range(3):
        a.forces.zero_()
        b.forces.zero_()
        _run(bp, lb, sets[1], out=b)
        g.replay()
        _run(bp, lb, sets[1], out=b)
        torch.cuda.synchronize()
        _same(a, ref[0])
        _same(b, ref[1])
