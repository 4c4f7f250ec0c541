"""The chemical potential against plain bisection on the host, over widths of the
Fermi function on which the launches' guesses of the root are good, useless, or
not made at all."""
import numpy as np
import pytest

from gpu_helpers import gpu_context, np_, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kT", [2.0, 0.1, 1e-3, 1e-5])
@pytest.mark.parametrize("filling", [0.002, 0.3, 0.999])
def test_mu_is_plain_bisections(kT, filling):
    import gen
    from scipy.special import expit
    torch_cuda()
    s = gen.make(1)
    ctx = gpu_context(s)
    ne = 8.0 * s.n_atoms * filling
    for tol in (1e-4, 1e-12):
        mu, _, _ = ctx.solve(nu=s.nu, kT=kT, n_electrons=ne, mu_tol=tol)
        eps, w, _ = (np_(x).ravel() for x in ctx.spectra())
        lo, hi, levels = eps[w != 0].min() - 40 * kT, eps[w != 0].max() + 40 * kT, 0
        while hi - lo > tol:
            mid = lo + (hi - lo) / 2
            if (w * expit((mid - eps) / kT)).sum() < ne:
                lo = mid
            else:
                hi = mid
            levels += 1
        f = expit((lo - eps) / kT)
        slope = (w * f * (1 - f)).sum() / kT
        # both sums over about 7,000 terms carry some 100 ulp of N_e, which moves
        # the root by that over dN/dmu; the two brackets may then be neighbours
        assert abs(mu - (lo + (hi - lo) / 2)) <= 1.01 * tol + 2.3e-14 * ne / slope
        assert ctx.stats()["bisect_levels"] == levels
