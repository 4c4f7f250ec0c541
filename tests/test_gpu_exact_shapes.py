"""The exact gradient with the forward pass in each of its workgroup shapes: the
kept basis, h, beta and last residual against differences of the grand potential
that the pass without them gives."""
import numpy as np
import pytest

from gpu_helpers import gpu_context, log, np_, torch_cuda
from test_gpu_grad import fd_forces
from test_gpu_krylov_shapes import _cluster_of_size

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nu", [12, 17, 20, 30])
@pytest.mark.parametrize("n", [64, 128, 160, 192])
def test_exact_forces_in_each_shape(nu, n):
    # the atom with the largest cluster, central differences with h = 1e-5 and
    # 2e-5 A and their Richardson combination, to 1e-6 eV/A as on the benchmark
    # cell.  The columns' bits do not depend on what is kept
    import gen
    torch_cuda()
    s = gen.make("mini_vac", nu=nu)
    J, s.r_cluster = _cluster_of_size(s, n)
    ctx = gpu_context(s)
    kw = dict(nu=nu, kT=s.kT, n_electrons=s.n_electrons)
    ctx.solve(**kw)
    plain = [np_(x) for x in ctx.spectra()]
    mu, _, _ = ctx.solve(keep_exact=True, **kw)
    for x, y in zip(plain, ctx.spectra()):
        assert np.array_equal(x, np_(y))
    F = np_(ctx.forces_exact(ctx._sk))[J]
    F1 = fd_forces(ctx, s, [J], mu, h=1e-5)[0]
    F2 = fd_forces(ctx, s, [J], mu, h=2e-5)[0]
    d = np.abs(F - (4.0 * F1 - F2) / 3.0).max()
    log(f"[exact shapes] nu {nu}, clusters up to {n} atoms: {d:.2e} eV/A")
    assert d <= 1e-6
