"""Krylov columns at the edges of the workgroup shapes: clusters that just fill
a shape's rows, exceed the shape below by one atom, or leave a tile of four
atoms ragged, at each basis capacity."""
import numpy as np
import pytest

from gpu_helpers import gpu_context, log, np_, torch_cuda

pytestmark = pytest.mark.gpu

SIZES = (17, 64, 65, 128, 129, 160, 161, 192)


def _cluster_of_size(s, n):
    """The atom with the tightest n nearest atoms (itself included) and a radius
    at which it has exactly n and no other atom has more."""
    d = s.pos[:, None, :] - s.pos[None, :, :]
    d -= s.cell * np.rint(d / s.cell)
    r = np.sort(np.sqrt((d ** 2).sum(-1)), axis=1)
    return int(np.argmin(r[:, n - 1])), 0.5 * (r[:, n - 1].min() + r[:, n].min())


@pytest.mark.parametrize("nu", [12, 20, 21, 30, 40, 48])
def test_columns_at_the_shape_edges(nu, monkeypatch):
    # eps to 1e-9: h and s carry about nu eps |H| = 48 x 2.2e-16 x 60 eV = 6e-13,
    # a well conditioned pencil (cond(s) below 1e3) brings at most 6e-10 of it
    # into eps; the weights, of order one, a tenth of that in absolute terms
    import gen
    from oracle import krylov, neighbors
    torch_cuda()
    s = gen.make("mini_vac")
    worst = [0.0, 0.0]
    for n in SIZES:
        J, s.r_cluster = _cluster_of_size(s, n)
        cols = 4 * J + np.arange(4, dtype=np.int32)
        ctx = gpu_context(s)
        eps, w, ne = (np_(x) for x in ctx.column_spectra(cols, nu=nu))
        clus = neighbors.cluster_of(s.pos, s.cell, J, s.r_cluster)
        assert clus.size == n
        Hc, Sc = neighbors.cluster_matrices(s.pos, s.cell, clus)
        l0 = 4 * int(np.searchsorted(clus, J))
        for i in range(4):
            ref = krylov.column_mode_k(Hc, Sc, l0 + i, nu)
            assert ne[i] == ref.nu_eff == nu
            worst[0] = max(worst[0], float(np.abs(eps[i] - ref.eps).max()))
            worst[1] = max(worst[1], float(np.abs(w[i] - ref.w).max()))
        # a column's bits depend neither on its partner nor on the LDS cache
        with monkeypatch.context() as m:
            m.setenv("MAG_LDS_CACHE", "0")  # read when a context makes its plans
            bare = gpu_context(s)
            for c, pick in ((ctx, [1]), (ctx, [3, 0]), (bare, [0, 1, 2, 3]), (bare, [2])):
                got = [np_(x) for x in c.column_spectra(cols[pick], nu=nu)]
                assert np.array_equal(got[0], eps[pick]) and np.array_equal(got[1], w[pick])
                assert np.array_equal(got[2], ne[pick])
    log(f"[shape edges nu {nu}] |d eps| {worst[0]:.2e} |d w| {worst[1]:.2e}")
    assert worst[0] <= 1e-9 and worst[1] <= 1e-10
