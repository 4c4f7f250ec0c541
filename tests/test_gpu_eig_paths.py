"""The two ways to run the projected eigensolves: a wave for each column up to
4,096 columns, a lane for each beyond."""
import numpy as np
import pytest

from gpu_helpers import gpu_context, np_, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nu", [3, 12, 20, 29, 40, 48])
def test_wave_and_lane_eigensolves_give_the_same_bits(nu):
    # both run the same QL steps, written without contraction: no tolerance
    import gen
    torch_cuda()
    s = gen.make(2)
    s.r_cluster = 3.0
    ctx = gpu_context(s)
    lane = [np_(x) for x in ctx.column_spectra(np.arange(4097, dtype=np.int32), nu=nu)]
    for first, last in ((0, 4096), (4096, 4097), (77, 142)):
        wave = [np_(x) for x in ctx.column_spectra(np.arange(first, last, dtype=np.int32), nu=nu)]
        for x, y in zip(wave, lane):
            assert np.array_equal(x, y[first:last])
