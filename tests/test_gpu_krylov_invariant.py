"""Columns whose Krylov space becomes invariant early beside a partner of the same
atom that goes on, in every workgroup shape: the second orthogonalization, after
which the column ends, or goes on along what is left."""
import numpy as np
import pytest

from gpu_helpers import gpu_context, log, np_, torch_cuda
from test_gpu_krylov_shapes import _cluster_of_size

pytestmark = pytest.mark.gpu


def _split_pencil(s, J, orb, delta, csr):
    """H and S on the pattern of `csr` with S = I and orbital `orb` of every atom
    coupled to that orbital alone, those of J and its three nearest atoms to the
    others' only by the fraction `delta`."""
    rowptr, colind, H, S = (np_(x) for x in csr)
    row = np.repeat(np.arange(rowptr.size - 1), np.diff(rowptr))
    d = s.pos - s.pos[J]
    d -= s.cell * np.rint(d / s.cell)
    group = np.zeros(s.n_atoms, dtype=bool)
    group[np.argsort((d ** 2).sum(-1))[:4]] = True
    own, other = row % 4 == orb, colind % 4 == orb
    H = np.where(own != other, 0.0, H)
    H = np.where(own & other & (group[row // 4] != group[colind // 4]), delta * H, H)
    return H, np.where(row == colind, 1.0, 0.0)


@pytest.mark.parametrize("orb", [0, 1])
@pytest.mark.parametrize("nu", [12, 20, 30, 40, 48])
def test_a_column_that_ends_early_leaves_its_partner_alone(nu, orb):
    # delta = 0: column `orb` is invariant after four steps.  delta = 1e-22: what
    # the second orthogonalization leaves is far above the breakdown bar and the
    # column goes on outside the four atoms.  eps to 1e-9 and w to 1e-10 as at the
    # shapes' edges (the pencil is orthonormal here, cond(s) = 1)
    import gen
    from oracle import krylov, neighbors
    torch_cuda()
    s = gen.make("mini_vac")
    for n in (64, 128, 160, 192):
        J, s.r_cluster = _cluster_of_size(s, n)
        ctx = gpu_context(s)
        cols = 4 * J + np.arange(4, dtype=np.int32)
        clus = neighbors.cluster_of(s.pos, s.cell, J, s.r_cluster)
        l0 = 4 * int(np.searchsorted(clus, J))
        ix = (4 * clus[:, None] + np.arange(4)).ravel()
        for delta, breakdown, dim in ((0.0, 1e-12, 4), (1e-22, 1e-30, nu)):
            H, S = _split_pencil(s, J, orb, delta, ctx._csr)
            ctx.update_values(H, S)
            dense = np.zeros((4 * s.n_atoms, 4 * s.n_atoms))
            rowptr, colind = np_(ctx._csr[0]), np_(ctx._csr[1])
            dense[np.repeat(np.arange(rowptr.size - 1), np.diff(rowptr)), colind] = H
            Hc, Sc = dense[np.ix_(ix, ix)], np.eye(ix.size)
            eps, w, ne = (np_(x) for x in ctx.column_spectra(cols, nu=nu, breakdown=breakdown))
            for i in range(4):
                ref = krylov.column_mode_k(Hc, Sc, l0 + i, nu, breakdown=breakdown)
                assert ne[i] == ref.nu_eff == (dim if i == orb else nu), (n, delta, i)
                assert np.abs(eps[i, :ne[i]] - ref.eps).max() <= 1e-9, (n, delta, i)
                assert np.abs(w[i, :ne[i]] - ref.w).max() <= 1e-10, (n, delta, i)
            for pick in ([orb], [1 - orb], [2, 3], [3, 1, orb]):
                got = [np_(x) for x in ctx.column_spectra(cols[pick], nu=nu, breakdown=breakdown)]
                for x, y in zip(got, (eps, w, ne)):
                    assert np.array_equal(x, y[pick]), (n, delta, pick)
            if nu <= 30:  # the kernel that also keeps the basis: the same columns
                kw = dict(nu=nu, kT=s.kT, n_electrons=s.n_electrons, breakdown=breakdown)
                for keep in (False, True):
                    ctx.solve(keep_exact=keep, **kw)
                    for x, y in zip((np_(x) for x in ctx.spectra()), (eps, w, ne)):
                        assert np.array_equal(x[cols], y), (n, delta, keep)
    log(f"[invariant nu {nu}] orbital {orb}: sizes 64 to 192")
