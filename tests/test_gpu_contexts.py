"""GPU: many contexts at a time (more than share one allocation of pinned
memory), and contexts made, used and destroyed by several threads: each
build's sizes and results are those of a context by itself."""
import threading

import numpy as np
import pytest

from paper_1812_07313_amd import bhq, synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _input(n):
    return tuple(torch.from_numpy(a).cuda() for a in synth.plummer(n, synth.rng(n)))


def _forces(ctx, x, m):
    bhq.bhq_set_eps(ctx, 0.01)
    bhq.bhq_build_lists_device(ctx, x, m, 0.7, 64)
    bhq.bhq_compute(ctx)
    return bhq.bhq_get_lists_sizes(ctx), bhq.bhq_get_result(ctx, len(m))[0]


def test_seventy_contexts():
    inputs = [_input(200 + 37 * (k % 5)) for k in range(5)]
    ctxs = []
    try:
        want = []
        for x, m in inputs:
            c = bhq.bhq_create(0, bhq.QUAD, bhq.FP32_OFS64)
            want.append(_forces(c, x, m))
            bhq.bhq_destroy(c)
        for _ in range(2):
            while len(ctxs) < 70:
                ctxs.append(bhq.bhq_create(0, bhq.QUAD, bhq.FP32_OFS64))
            for k, c in enumerate(ctxs):
                sizes, a = _forces(c, *inputs[k % 5])
                assert sizes == want[k % 5][0] and np.array_equal(a, want[k % 5][1])
            for c in ctxs[10:60]:
                bhq.bhq_destroy(c)
            ctxs = ctxs[:10] + ctxs[60:]
    finally:
        for c in ctxs:
            bhq.bhq_destroy(c)


def test_contexts_of_threads():
    inputs = [_input(300 + 100 * k) for k in range(8)]
    want = []
    for x, m in inputs:
        c = bhq.bhq_create(0, bhq.QUAD, bhq.FP32_OFS64)
        want.append(_forces(c, x, m))
        bhq.bhq_destroy(c)
    bad = []

    def work(k):
        try:
            for _ in range(20):
                c = bhq.bhq_create(0, bhq.QUAD, bhq.FP32_OFS64)
                try:
                    sizes, a = _forces(c, *inputs[k])
                finally:
                    bhq.bhq_destroy(c)
                if sizes != want[k][0] or not np.array_equal(a, want[k][1]):
                    bad.append(k)
        except Exception as e:  # noqa: BLE001 - reported below
            bad.append((k, e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad
