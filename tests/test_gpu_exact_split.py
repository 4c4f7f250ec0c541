"""The exact gradient by single columns (up to four atoms per CU) against whole
atoms (beyond): the same force parts, added in the same order."""
import numpy as np
import pytest

from gpu_helpers import gpu_context, np_, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nu", [12, 20, 30])
def test_translated_copies_get_the_same_forces_by_columns_and_by_atoms(nu):
    # one cell of 3,892 atoms (whole atoms) against the forces on its atoms that
    # the same clusters give in a cell of 487 atoms repeated 2 x 2 x 2: at equal
    # mu every atom's clusters are equal, so only rounding is left.  Each force
    # adds about 150 parts of at most 1 eV/A whose columns carry some 1e-13:
    # 1e-10 with three orders for the conditioning of the pencils
    import gen
    torch = torch_cuda()
    s = gen.make("mini_vac")
    s.r_cluster = 4.2
    small = gpu_context(s)
    kw = dict(nu=nu, kT=s.kT, mu_fixed=3.0)
    small.solve(n_electrons=s.n_electrons, **kw)
    F1 = np_(small.forces_exact(small._sk))
    shifts = np.stack(np.meshgrid(*[np.arange(2)] * 3, indexing="ij"), -1).reshape(-1, 3)
    s.pos = (s.pos[None] + shifts[:, None] * s.cell).reshape(-1, 3)
    s.cell = 2.0 * s.cell
    big = gpu_context(s)
    big.solve(n_electrons=8 * s.n_electrons, **kw)
    F8 = np_(big.forces_exact(big._sk)).reshape(8, -1, 3)
    assert small._pos.shape[0] <= 1024 < big._pos.shape[0]
    assert np.abs(F8 - F1).max() <= 1e-10
