"""The grid schedule takes one, two or four columns of an atom per workgroup: the
same bits as the persistent one, also where the list breaks an atom's columns up."""
import numpy as np
import pytest

from gpu_helpers import gpu_context, np_, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nu", [12, 40])
def test_grid_and_persistent_columns_are_the_same(nu):
    import gen
    torch_cuda()
    s = gen.make(2)
    s.r_cluster = 3.0
    ctx = gpu_context(s)
    every = np.arange(4 * s.n_atoms, dtype=np.int32)
    shuffled = np.random.default_rng(5).permutation(every)
    for cols in (every[:1], every[2:5], every[:801], every[1:1602], every, every[::3], shuffled):
        want = ctx.column_spectra(cols, nu=nu, schedule="persistent")
        for x, y in zip(ctx.column_spectra(cols, nu=nu, schedule="grid"), want):
            assert np.array_equal(np_(x), np_(y))
