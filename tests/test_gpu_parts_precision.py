"""GPU: the parts that a context chooses have memory per precision, and a change
of precision (also while a stream is captured) moves none of it."""
import numpy as np
import pytest

from paper_1812_07313_amd import bhq, synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N = 4096  # one list of few groups: parts


def _context(precision, n=N, seed=46):
    x, m = (torch.from_numpy(a).cuda() for a in synth.plummer(n, synth.rng(seed)))
    ctx = bhq.bhq_create(0, bhq.QUAD, precision)
    bhq.bhq_set_eps(ctx, 0.01)
    bhq.bhq_build_lists_device(ctx, x, m, 0.6, 64)
    return ctx


def _forces(ctx, n=N):
    """Of bhq_compute and of bhq_compute_noalloc."""
    bhq.bhq_compute(ctx)
    a = torch.zeros(n, 3, dtype=torch.float64, device="cuda")
    bhq.bhq_compute_noalloc(ctx, a, None)
    torch.cuda.synchronize()
    return bhq.bhq_get_result(ctx, n)[0], a.cpu().numpy()


@pytest.mark.parametrize("first", [bhq.FP32_OFS64, bhq.FP64])
def test_switch(first):
    """Forth and back, and on longer lists: the bits of contexts that were made
    for the precision."""
    want = {}
    for n, seed in ((N, 46), (2 * N + 77, 47)):
        for prec in (bhq.FP32_OFS64, bhq.FP64):
            c = _context(prec, n, seed)
            want[n, prec] = _forces(c, n)
            bhq.bhq_destroy(c)
    second = bhq.FP64 if first == bhq.FP32_OFS64 else bhq.FP32_OFS64
    ctx = _context(first)
    try:
        for n, seed in ((N, 46), (2 * N + 77, 47), (N, 46)):
            x, m = (torch.from_numpy(a).cuda() for a in synth.plummer(n, synth.rng(seed)))
            bhq.bhq_build_lists_device(ctx, x, m, 0.6, 64)
            for prec in (first, second, first):
                bhq.bhq_set_kernel(ctx, bhq.QUAD, prec)
                for got, w in zip(_forces(ctx, n), want[n, prec]):
                    assert np.array_equal(got, w)
    finally:
        bhq.bhq_destroy(ctx)


def test_switch_while_capturing():
    """The FP32 evaluation captured before the change and the FP64 one after it
    replay side by side."""
    ctx = _context(bhq.FP32_OFS64)
    try:
        want32 = _forces(ctx)[1]
        c = _context(bhq.FP64)
        want64 = _forces(c)[1]
        bhq.bhq_destroy(c)
        a32 = torch.zeros(N, 3, dtype=torch.float64, device="cuda")
        a64 = torch.zeros_like(a32)
        s = torch.cuda.Stream()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            bhq.bhq_compute_noalloc(ctx, a32, None, stream=s)
            bhq.bhq_set_kernel(ctx, bhq.QUAD, bhq.FP64)
            bhq.bhq_compute_noalloc(ctx, a64, None, stream=s)
        for _ in range(3):
            a32.zero_(), a64.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(a32.cpu().numpy(), want32)
            assert np.array_equal(a64.cpu().numpy(), want64)
            bhq.bhq_compute(ctx)
    finally:
        torch.cuda.synchronize()
        bhq.bhq_destroy(ctx)
