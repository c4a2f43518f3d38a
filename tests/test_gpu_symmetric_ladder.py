"""The FP64 ladder of symmetric vertices (k_ladder_screen + k_ladder_sym) and its
dispatch against the oracle, at every tile-count boundary of n_nu.

Tolerances are the FP64 path's: max|Delta| / max|ref| <= 1e-12 on W, 1e-11 on
log det, status bit-exact.
"""
import numpy as np
import pytest

from oracle import df_oracle as O
from paper_1507_00895_amd import inputs as I

pytestmark = pytest.mark.gpu

TOL_W, TOL_LD = 1e-12, 1e-11


def solve(p, symmetry=0):
    import torch
    from paper_1507_00895_amd import binding as B
    inst = B.make_instance(p)
    opts = B.make_opts(symmetry=symmetry)
    ws = B.workspace([inst], opts)
    B.df_dual_gf([inst], ws)
    B.df_bubble([inst], ws)
    B.df_ladder_solve([inst], ws, opts)
    torch.cuda.synchronize()
    return inst


def check(p, inst):
    lr = O.ladder(O.spin_channels(p.gamma_uu, p.gamma_ud), inst.chi.cpu().numpy())
    assert np.array_equal(inst.status.cpu().numpy(), lr.status)
    w, ld = inst.w.cpu().numpy(), inst.logdet.cpu().numpy()
    assert np.abs(w - lr.W).max() / np.abs(lr.W).max() <= TOL_W
    ok = lr.status != 2
    assert np.abs(ld.real - lr.logdet.real)[ok].max() <= TOL_LD
    assert np.abs(np.exp(1j * ld.imag) - np.exp(1j * lr.logdet.imag))[ok].max() <= TOL_LD
    return lr


def symmetric_problem(D, nk, n_nu, n_om, seed, scale=0.6):
    """Dense complex vertex, symmetric in its frequencies, max |gamma chi| row sum
    near `scale` (certified everywhere)."""
    p = I.atomic_limit_problem(D, nk, n_nu, n_om, 10.0, 2.0, 0.1)
    rng = np.random.default_rng(seed)
    chi = O.bubble_fft(O.dual_gf0(p.g, p.delta, p.eps), D, nk, n_om, p.beta)
    gs = []
    for _ in range(2):
        a = rng.standard_normal((n_om, n_nu, n_nu)) + 1j * rng.standard_normal((n_om, n_nu, n_nu))
        gs.append(a + a.transpose(0, 2, 1))
    rows = max(float((np.abs(g[m])[None] * np.abs(chi[m]).T[:, None, :]).sum(2).max())
               for g in (gs[0] + gs[1], gs[0] - gs[1]) for m in range(n_om))
    p.gamma_uu, p.gamma_ud = (scale / rows * g for g in gs)
    return p


# one below, at and above every multiple of 16 (n_nu is even), and the extremes
SIZES = [2, 14, 16, 18, 30, 32, 34, 46, 48, 50, 62, 64, 66, 78, 80, 82, 94, 96, 98, 110, 112, 114, 126, 128]


@pytest.mark.parametrize("n_nu", SIZES)
def test_symmetric_vertex_sizes(n_nu):
    p = symmetric_problem(1, 8, n_nu, min(3, n_nu - 1), seed=n_nu)
    lr = check(p, solve(p))
    assert (lr.status == 0).all()


@pytest.mark.parametrize("n_nu", [16, 48, 64, 96, 128])
def test_antisymmetric_part_at_rounding_level_drops_out(n_nu):
    """An antisymmetric part of 5e-13 max|gamma| still runs the symmetric kernel;
    its first-order effect on Gamma_nn and log det vanishes."""
    p = symmetric_problem(1, 8, n_nu, 3, seed=1000 + n_nu)
    rng = np.random.default_rng(n_nu)
    for name in ("gamma_uu", "gamma_ud"):
        g = getattr(p, name)
        a = rng.uniform(-1, 1, g.shape) + 1j * rng.uniform(-1, 1, g.shape)
        big = min(np.abs(p.gamma_uu + p.gamma_ud).max((1, 2)).min(), np.abs(p.gamma_uu - p.gamma_ud).max((1, 2)).min())
        setattr(p, name, g + 6e-14 * big * (a - a.transpose(0, 2, 1)))
    check(p, solve(p))


@pytest.mark.parametrize("n_nu", [14, 48, 66, 96])
def test_mixed_symmetric_and_general_vertices(n_nu):
    """One bosonic frequency's vertex is not symmetric: its items take the general
    kernel in the same call, alone and fused with a symmetric instance."""
    import torch
    from paper_1507_00895_amd import binding as B
    p = symmetric_problem(1, 8, n_nu, 3, seed=2000 + n_nu)
    rng = np.random.default_rng(n_nu)
    p.gamma_uu = p.gamma_uu.copy()
    p.gamma_uu[2] += 0.1 * np.abs(p.gamma_uu[2]).max() * rng.uniform(-1, 1, (n_nu, n_nu))
    check(p, solve(p))
    q = symmetric_problem(2, 4, n_nu, 1, seed=3000 + n_nu)
    insts = [B.make_instance(x) for x in (p, q)]
    ws = B.workspace(insts)
    B.df_dual_gf(insts, ws)
    B.df_bubble(insts, ws)
    B.df_ladder_solve(insts, ws)
    torch.cuda.synchronize()
    for x, inst in zip((p, q), insts):
        check(x, inst)


@pytest.mark.parametrize("n_nu", [18, 64, 82, 128])
def test_items_outside_the_certificate(n_nu):
    """Coupling up to and beyond the radius: uncertified items are pivoted, the
    others stay in the symmetric kernel."""
    p = symmetric_problem(1, 16, n_nu, 3, seed=4000 + n_nu, scale=2.5)
    check(p, solve(p))


@pytest.mark.parametrize("n_nus", [(66, 72, 80), (98, 104, 128)])
def test_fused_instances_of_one_padded_size(n_nus):
    """Instances whose n_nu differ but shared one launch class before: each has its
    own number of 16-row blocks."""
    import torch
    from paper_1507_00895_amd import binding as B
    ps = [symmetric_problem(1, 8, n, 3, seed=n) for n in n_nus]
    insts = [B.make_instance(p) for p in ps]
    ws = B.workspace(insts)
    B.df_dual_gf(insts, ws)
    B.df_bubble(insts, ws)
    B.df_ladder_solve(insts, ws)
    torch.cuda.synchronize()
    for p, inst in zip(ps, insts):
        check(p, inst)


def test_nonfinite_inputs_are_flagged():
    """A NaN or infinity in chi makes its own items non-finite (status 2) and no others."""
    import torch
    from paper_1507_00895_amd import binding as B
    p = symmetric_problem(1, 16, 48, 3, seed=5)
    inst = B.make_instance(p)
    ws = B.workspace([inst])
    B.df_dual_gf([inst], ws)
    B.df_bubble([inst], ws)
    inst.chi[1, 5, 3] = float("nan")
    inst.chi[1, 40, 9] = float("inf")
    B.df_ladder_solve([inst], ws)
    torch.cuda.synchronize()
    st = inst.status.cpu().numpy()
    want = np.zeros_like(st)
    want[:, 1, 3] = want[:, 1, 9] = 2
    assert np.array_equal(st, want)
    assert np.isfinite(inst.w.cpu().numpy()[:, [0, 2]]).all()
