"""FP64 ladder of vertices that are not symmetric in their frequencies (what a measured
vertex is, to its noise) against the oracle: at the edges of every padded size, certified
everywhere and with uncertified items among them, and in launches of several rounds of
the grid.

Tolerances are the FP64 path's: max|Delta| / max|ref| <= 1e-12 on W, 1e-11 on
log det, status bit-exact.
"""
import numpy as np
import pytest

from oracle import df_oracle as O
from paper_1507_00895_amd import inputs as I

pytestmark = pytest.mark.gpu

TOL_W, TOL_LD = 1e-12, 1e-11


def problem(D, nk, n_nu, n_om, scale):
    """Dense complex vertex, max |gamma chi| row sum `scale`."""
    p = I.atomic_limit_problem(D, nk, n_nu, n_om, 10.0, 2.0, 0.1)
    rng = np.random.default_rng(n_nu)
    chi = O.bubble_fft(O.dual_gf0(p.g, p.delta, p.eps), D, nk, n_om, p.beta)
    gs = [rng.standard_normal((n_om, n_nu, n_nu)) + 1j * rng.standard_normal((n_om, n_nu, n_nu))
          for _ in range(2)]
    rows = max(float((np.abs(g[m]) @ np.abs(chi[m])).max())
               for g in (gs[0] + gs[1], gs[0] - gs[1]) for m in range(n_om))
    p.gamma_uu, p.gamma_ud = (scale / rows * g for g in gs)
    return p


def solve(p, chi=None, **opts):
    import torch
    from paper_1507_00895_amd import binding as B
    inst = B.make_instance(p)
    o = B.make_opts(**opts)
    ws = B.workspace([inst], o)
    if chi is None:
        B.df_dual_gf([inst], ws)
        B.df_bubble([inst], ws)
    else:
        inst.chi.copy_(torch.as_tensor(chi))
    B.df_ladder_solve([inst], ws, o)
    torch.cuda.synchronize()
    return inst


def check(w, ld, st, ref):
    assert np.array_equal(st, ref.status)
    assert np.abs(w - ref.W).max() / np.abs(ref.W).max() <= TOL_W
    assert np.abs(ld.real - ref.logdet.real).max() <= TOL_LD
    assert np.abs(np.exp(1j * ld.imag) - np.exp(1j * ref.logdet.imag)).max() <= TOL_LD


# (n_nu, nk of a 2D grid, n_om): launches above the item counts of the sizes' small-launch
# route (2560 waves, 32768 items of one wave each) and below them
SHAPES = [(14, 64, 5), (16, 64, 5), (18, 32, 3), (32, 32, 3), (34, 16, 3), (48, 16, 3),
          (50, 16, 3), (62, 16, 3), (64, 16, 3), (66, 16, 1), (80, 8, 3), (94, 8, 3), (96, 8, 3),
          (98, 8, 3), (112, 8, 1), (126, 8, 1), (128, 8, 1),
          (2, 64, 1), (2, 4, 1), (14, 8, 3), (16, 32, 5), (32, 8, 3), (48, 8, 3), (50, 8, 3), (64, 8, 3)]


@pytest.mark.parametrize("scale", [0.6, 2.5])
@pytest.mark.parametrize("n_nu,nk,n_om", SHAPES)
def test_general_vertex(n_nu, nk, n_om, scale):
    p = problem(2, nk, n_nu, n_om, scale)
    inst = solve(p)
    ref = O.ladder(O.spin_channels(p.gamma_uu, p.gamma_ud), inst.chi.cpu().numpy())
    if scale < 1:
        assert (ref.status == 0).all()
    check(inst.w.cpu().numpy(), inst.logdet.cpu().numpy(), inst.status.cpu().numpy(), ref)


@pytest.mark.parametrize("n_nu,nk,n_om", [(96, 64, 3), (98, 64, 3), (128, 64, 9)])
def test_launches_of_many_rounds(n_nu, nk, n_om):
    """More items than the grid (at n_nu 128 more than 64 rounds of it): a sample of the
    momenta, the last ones among them."""
    p = problem(2, 8, n_nu, n_om, 0.6)
    q = I.atomic_limit_problem(2, nk, n_nu, n_om, 10.0, 2.0, 0.1)
    rng = np.random.default_rng(1)
    # the bubble of the small grid at random momenta of the large one: bounded row sums
    small = O.bubble_fft(O.dual_gf0(p.g, p.delta, p.eps), 2, 8, n_om, p.beta)
    chi = np.ascontiguousarray(small[:, :, rng.integers(0, 64, nk * nk)])
    q.gamma_uu, q.gamma_ud = p.gamma_uu, p.gamma_ud
    inst = solve(q, chi)
    pick = np.concatenate([rng.integers(0, nk * nk, 4), [nk * nk - 2, nk * nk - 1]])
    ref = O.ladder(O.spin_channels(p.gamma_uu, p.gamma_ud), chi[:, :, pick])
    check(inst.w.cpu().numpy()[..., pick], inst.logdet.cpu().numpy()[..., pick],
          inst.status.cpu().numpy()[..., pick], ref)
    assert (inst.status.cpu().numpy() == 0).all() and np.isfinite(inst.w.cpu().numpy()).all()


@pytest.mark.parametrize("n_nu", [14, 48, 64, 96, 128])
def test_symmetry_reduced_and_refined(n_nu):
    """The reduced items of an instance, and the refined class, whose items near the
    instability take the same elimination, against FP64 without reduction."""
    from paper_1507_00895_amd import binding as B
    p = problem(2, 16, n_nu, 3, 0.97)
    a = solve(p)
    w = a.w.cpu().numpy()
    r = solve(p, prec=B.DF_FP32_REFINE)
    assert np.array_equal(r.status.cpu().numpy(), a.status.cpu().numpy())
    assert np.abs(r.w.cpu().numpy() - w).max() <= 1e-9 * np.abs(w).max()
    s = solve(p, symmetry=1)
    # Omega >= 0 and the orbits' representatives are solved, the rest is copied from them
    # (the vertex itself lacks the conjugation symmetry): momentum 0, Omega >= 0
    got = s.w.cpu().numpy()[:, 1:, :, 0]
    assert np.abs(got - w[:, 1:, :, 0]).max() <= TOL_W * np.abs(w).max()
