"""The FFT kernels on every supported grid shape (each is a build of its own) against
the oracle: dual propagator with its inverse transform, bubble, Schwinger-Dyson
convolution, on unstructured complex fields, with one and several bosonic
frequencies (frequencies that leave the window included).

Tolerance: the FP64 path's, max|Delta| / max|ref| <= 1e-12.
"""
import numpy as np
import pytest

from oracle import df_oracle as O
from paper_1507_00895_amd import inputs as I

pytestmark = pytest.mark.gpu

TOL = 1e-12
SHAPES = [(D, nk) for D in (1, 2, 3, 4) for nk in (4, 8, 16, 32, 64) if nk ** D <= 4096]


def rel(x, ref):
    return float(np.abs(x.cpu().numpy() - ref).max() / np.abs(ref).max())


@pytest.mark.parametrize("n_nu,n_om", [(2, 1), (6, 5), (64, 3)])
@pytest.mark.parametrize("D,nk", SHAPES)
def test_fft_kernels(D, nk, n_nu, n_om):
    import torch
    from paper_1507_00895_amd import binding as B
    p = I.atomic_limit_problem(D, nk, n_nu, n_om, 7.0, 2.0, 0.1)
    x = B.make_instance(p)
    ws = B.workspace([x])
    S = 0.1 * I.random_complex((n_nu, p.N), seed=D * 100 + nk)
    x.sigma.copy_(torch.as_tensor(S))
    B.df_dual_gf([x], ws)
    torch.cuda.synchronize()
    G = O.dual_gf(O.dual_gf0(p.g, p.delta, p.eps), S)
    assert rel(x.gd, G) <= TOL
    # unstructured fields: no symmetry hides a wrong reflection or axis order
    G = I.random_complex((n_nu, p.N), seed=nk + 1)
    W = I.random_complex((2, n_om, n_nu, p.N), seed=nk + 2)
    x.gd.copy_(torch.as_tensor(G))
    x.w.copy_(torch.as_tensor(W))
    B.df_bubble([x], ws)
    B.df_sigma([x], ws)
    torch.cuda.synchronize()
    assert rel(x.chi, O.bubble_fft(G, D, nk, n_om, p.beta)) <= TOL
    assert rel(x.sigma_calc, O.sigma_fft(W, G, D, nk, p.beta)) <= TOL
    # the fused sequence of the loop: dual propagator and its transform in one kernel
    x.sigma.copy_(torch.as_tensor(S))
    B.df_iterate([x], ws, B.make_opts(mix=1.0, max_iter=1), allow=(B.DF_OK, B.DF_W_FALLBACK))
    G = O.dual_gf(O.dual_gf0(p.g, p.delta, p.eps), S)
    assert rel(x.chi, O.bubble_fft(G, D, nk, n_om, p.beta)) <= TOL
