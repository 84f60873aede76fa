"""A batch that was captured once still enqueues calls with unchanged arrays on
alternating streams without waiting for the device: work of a stream that has
nothing to do with the batch is still running when they return."""
import pytest

from test_gpu_batch_buffers import _inputs, _plan, _run, _same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lb", [False, True], ids=["geometric", "lb"])
def test_unchanged_arrays_on_two_streams_after_a_capture(lb):
    import torch
    x = _inputs(1, lb)
    bp = _plan(lb)
    bp.set_graph(False)
    out = _run(bp, lb, x)
    torch.cuda.synchronize()
    ref = _run(_plan(lb), lb, x)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        _run(bp, lb, x, out=out)
    m = torch.randn(8192, 8192, device="cuda")
    r = torch.empty_like(m)
    streams = [torch.cuda.Stream() for _ in range(3)]
    with torch.cuda.stream(streams[0]):
        _run(bp, lb, x, out=out)
    torch.mm(m, m, out=r)
    torch.cuda.synchronize()
    busy = torch.cuda.Event()
    with torch.cuda.stream(streams[2]):
        for _ in range(60):   # some 0.5 s
            torch.mm(m, m, out=r)
        busy.record()
    for k in (1, 0, 1, 0):
        streams[k].wait_stream(streams[1 - k])
        with torch.cuda.stream(streams[k]):
            _run(bp, lb, x, out=out)
    assert not busy.query()
    torch.cuda.synchronize()
    _same(out, ref)
    g.replay()
    torch.cuda.synchronize()
    _same(out, ref)


@pytest.mark.parametrize("own", [False, True], ids=["second stream", "the capture's stream"])
def test_new_arrays_after_a_capture_wait_for_the_ones_in_flight(own):
    """An evaluation still waiting on its stream keeps its arrays when a call
    with others is captured and then made on another stream."""
    import torch
    x, y = _inputs(1, False), _inputs(2, False)
    bp = _plan(False)
    bp.set_graph(False)
    refx, refy = _run(_plan(False), False, x), _run(_plan(False), False, y)
    outx, outy = _run(bp, False, x), _run(bp, False, y)
    m = torch.randn(8192, 8192, device="cuda")
    r = torch.mm(m, m)
    a, b, c = (torch.cuda.Stream() for _ in range(3))
    torch.cuda.synchronize()
    outx.forces.zero_()
    outy.forces.zero_()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(a):
        for _ in range(30):
            torch.mm(m, m, out=r)
        _run(bp, False, y, out=outy)
    with torch.cuda.stream(c):
        g.capture_begin(capture_error_mode="relaxed")
        _run(bp, False, x, out=outx)
        g.capture_end()
    with torch.cuda.stream(c if own else b):
        _run(bp, False, x, out=outx)
    torch.cuda.synchronize()
    _same(outy, refy)
    _same(outx, refx)
