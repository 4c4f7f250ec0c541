"""Brackets of the chemical potential wider than the halvings granted are refused,
whatever the launches could decide."""
import pytest

from gpu_helpers import gpu_context, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("schedule", ["persistent", "graph"])
def test_brackets_beyond_the_granted_halvings_are_refused(schedule):
    # at half filling mu lies among the levels however wide the bracket of 80 kT.
    # tol = 1e-4 grants 40 halvings: 80 kT / 2^40 <= tol up to kT = 1.37e6 eV
    import gen
    from paper_1210_1531_amd import MagError, _lib as L
    torch_cuda()
    s = gen.make(1)
    ctx = gpu_context(s)
    kw = dict(nu=s.nu, n_electrons=4.0 * s.n_atoms, mu_tol=1e-4, schedule=schedule)
    ctx.solve(kT=1.3e6, **kw)
    for _ in range(3):  # (with a graph: eagerly, captured, replayed)
        with pytest.raises(MagError) as e:
            ctx.solve(kT=2e6, **kw)
        assert e.value.status == L.MAG_EBRACKET
    ctx.solve(kT=1.3e6, **kw)
