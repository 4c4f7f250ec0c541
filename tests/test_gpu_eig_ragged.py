"""The projected eigensolves of columns whose Krylov spaces end early, by lanes and
by waves."""
import numpy as np
import pytest

from gpu_helpers import gpu_context, np_, torch_cuda

pytestmark = pytest.mark.gpu


def test_wave_and_lane_eigensolves_agree_on_ragged_columns():
    # perfect diamond with 10% vacancies and five-atom clusters: 3 to 13 steps a
    # column, no two neighbours need the same.  Both ways run the same QL steps: no
    # tolerance.  More columns than run by waves, then pieces that do
    from gen import structures as gs
    torch_cuda()
    s = gs.make_structure(cells=(6, 6, 6), vacancy_frac=0.1, sigma=0.0, seed=4, nu=30,
                          r_cluster=2.0, name="vac_nn")
    ctx = gpu_context(s, sk=dict(r_on=1.7, r_cut=1.8))
    kw = dict(nu=s.nu, breakdown=1e-8)
    m = 4 * s.n_atoms
    assert m > 4096
    lane = [np_(x) for x in ctx.column_spectra(np.arange(m, dtype=np.int32), **kw)]
    assert np.unique(lane[2]).size >= 5 and lane[2].max() < s.nu
    for first, last in ((0, 2000), (2000, 4096), (4096, m), (m - 1, m)):
        wave = [np_(x) for x in ctx.column_spectra(np.arange(first, last, dtype=np.int32), **kw)]
        for x, y in zip(wave, lane):
            assert np.array_equal(x, y[first:last])
