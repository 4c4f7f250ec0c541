"""The chemical potential where N(mu) is not monotone: truncated columns of a
generalized problem have some negative weights, and at small kT N falls across
such a level.  Electron counts inside the falls have several roots."""
import numpy as np
import pytest

from gpu_helpers import gpu_context, np_, torch_cuda

pytestmark = pytest.mark.gpu


def _fillings_in_falls(eps, w, kT, count=3):
    """(lowest, highest) N of each fall next to a negative weight, and `count`
    electron counts inside it."""
    from scipy.special import expit
    out = []
    for e0 in eps[w < 0]:
        x = e0 + kT * np.linspace(-12, 12, 193)
        n = (w * expit((x[:, None] - eps) / kT)).sum(1)
        i = np.flatnonzero(np.diff(n) < 0)
        if i.size:
            top, bottom = n[i[0]], n[i[-1] + 1]
            out += list(bottom + np.linspace(0.15, 0.95, count) * (top - bottom))
    return out


@pytest.mark.parametrize("nu", [30, 40])
@pytest.mark.parametrize("kT", [1e-2, 1e-3, 1e-4, 1e-5])
def test_mu_is_a_root_inside_the_falls_of_N(nu, kT):
    # |N(mu) - N_e| of the returned mu, and the halvings, must be plain
    # bisection's: 1e-9 of residual wherever plain bisection has that
    import gen
    from oracle import fermi
    torch_cuda()
    s = gen.make(1, nu=nu)
    ctx = gpu_context(s)
    ctx.solve(nu=nu, kT=kT, n_electrons=s.n_electrons)
    eps, w, _ = (np_(x).ravel() for x in ctx.spectra())
    eps, w = eps[w != 0], w[w != 0]
    fillings = _fillings_in_falls(eps, w, kT)
    if (nu, kT) == (30, 1e-3):
        fillings.append(14.013013598616636)
    assert fillings or (nu, kT) == (30, 1e-2)  # (no fall is deep enough there)
    for ne in fillings:
        mu, _, _ = ctx.solve(nu=nu, kT=kT, n_electrons=float(ne))
        ref, levels = fermi.bisect_mu(eps, w, kT, ne)
        if abs(fermi.electron_count(ref, eps, w, kT) - ne) <= 1e-9:
            got = fermi.electron_count(mu, eps, w, kT) - ne
            assert abs(got) <= 1e-9, (ne, mu, ref, got)
        assert ctx.stats()["bisect_levels"] == levels
