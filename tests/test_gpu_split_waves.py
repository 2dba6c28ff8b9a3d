"""GPU: the FP32 split kernels' default launch caps registers for six waves only
where that pays: on few or small groups it is as fast as the launch without the
cap, on many ordinary ones faster, and the bits are the same."""
import numpy as np
import pytest

from paper_1812_07313_amd import bhq, synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _time(ctx):
    t, spent = [], 0.0
    while spent < 8.0:
        bhq.bhq_compute(ctx)
        t.append(bhq.bhq_get_kernel_ms(ctx))
        spent += t[-1]
    return min(t[len(t) // 2:])


@pytest.mark.parametrize("kernel", [bhq.SPLIT_QUAD, bhq.SPLIT_MONO])
@pytest.mark.parametrize("side,ncrit,ratio", [(12, 16, 1.08), (16, 16, 1.08), (24, 256, 1.08),
                                              (48, 16, 1.08), (64, 256, 0.98)])
def test_default_against_uncapped(kernel, side, ncrit, ratio):
    """Capped for six waves, the first four took 1.05 to 1.6 times as long; the
    last takes 0.93 of the time with the cap."""
    n, rs = side ** 3, 1.25 / side
    x, m = (torch.from_numpy(a).cuda() for a in synth.perturbed_lattice(side, synth.rng(1)))
    default, plain = (bhq.bhq_create(0, kernel, bhq.FP32_OFS64) for _ in range(2))
    out, ms = {}, {}
    try:
        for c in (default, plain):
            bhq.bhq_set_split(c, rs, 4.5 * rs, 1.0)
            bhq.bhq_build_lists_device(c, x, m, 0.5, ncrit, 8, 1.0, 4.5 * rs)
        for _ in range(3):
            for name, c, waves in (("default", default, None), (0, plain, 0), (6, plain, 6)):
                if waves is not None:
                    bhq.bhq_set_tuning(c, 256, 2, waves_per_eu=waves)
                ms[name] = min(ms.get(name, np.inf), _time(c))
                out[name] = bhq.bhq_get_result(c, n)
    finally:
        bhq.bhq_destroy(default)
        bhq.bhq_destroy(plain)
    for waves in (0, 6):
        assert all(np.array_equal(a, b) for a, b in zip(out["default"], out[waves]))
    assert ms["default"] < ratio * ms[0], ms
