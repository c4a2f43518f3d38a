"""df_lattice on a vertex that counts as symmetric but is not exactly so, at couplings up to
and beyond the radius: the uncertified items' elimination takes the same (symmetrised)
vertex in its matrix and its right-hand side.

With one vertex S = (gamma + gamma^T) / 2 throughout, the antisymmetric part enters in second
order (1e-24) and what is left is the rounding of S, 1.1e-16 per element, times the
ladder's amplification (condition about 1e2): 2e-14 between the observables of gamma and of
S.  With S in one place and gamma in the other it enters in first order, 7e-14 to 5e-13.
"""
import numpy as np
import pytest

from test_gpu_lattice_ladder import problem, run

pytestmark = pytest.mark.gpu


def observables(p):
    import torch
    from paper_1507_00895_amd import binding as B
    x = B.make_instance(p, outputs=False)
    ch, sp = (torch.empty(p.N, dtype=torch.complex128, device="cuda") for _ in range(2))
    B.df_lattice(x, p.mu, None, None, ch, sp)
    torch.cuda.synchronize()
    return ch.cpu().numpy(), sp.cpu().numpy()


@pytest.mark.parametrize("n_nu", [16, 64, 98])
def test_antisymmetric_part_at_rounding_level_beyond_the_radius(n_nu):
    p = problem(n_nu, 400 + n_nu, 5.0)
    s = problem(n_nu, 400 + n_nu, 5.0)
    rng = np.random.default_rng(n_nu)
    big = min(np.abs(p.gamma_uu + p.gamma_ud).max(), np.abs(p.gamma_uu - p.gamma_ud).max())
    for name in ("gamma_uu", "gamma_ud"):
        a = rng.uniform(-1, 1, (1, n_nu, n_nu)) + 1j * rng.uniform(-1, 1, (1, n_nu, n_nu))
        g = getattr(p, name) + 6e-14 * big * (a - a.transpose(0, 2, 1))
        setattr(p, name, g)
        setattr(s, name, 0.5 * (g + g.transpose(0, 2, 1)))
    for got, want in zip(observables(p), observables(s)):
        assert np.abs(got - want).max() <= 2e-14 * np.abs(want).max()
    run(p)
