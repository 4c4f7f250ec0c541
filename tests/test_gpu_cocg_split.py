"""The ways to share COCG energies among workgroups (one, two or four each)."""
import numpy as np
import pytest

from gpu_helpers import gpu_context, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ncols,nz", [(193, 4), (155, 5), (385, 2), (769, 1)])
def test_energies_alone_and_together_give_the_same_bits(ncols, nz):
    # past 768 (column, energy) pairs energies share a workgroup; one energy's
    # arithmetic does not depend on it: no tolerance
    import gen
    torch_cuda()
    s = gen.make("mini_vac")
    s.r_cluster = 3.2
    ctx = gpu_context(s)
    cols = np.arange(ncols, dtype=np.int32)
    z = np.linspace(-6.0, 6.0, nz) + 0.7j
    G, off, it = ctx.cocg_columns(cols, z)
    pick = np.array([0, 1, ncols // 2, ncols - 1], dtype=np.int32)
    for q in range(nz):
        g1, off1, it1 = ctx.cocg_columns(pick, z[q:q + 1])
        for i, j in enumerate(pick):
            n = off[j + 1] - off[j]
            whole = G[off[j] * nz + q * n:off[j] * nz + (q + 1) * n]
            assert np.array_equal(g1[off1[i]:off1[i + 1]], whole)
            assert it1[i, 0] == it[j, q] > 0
