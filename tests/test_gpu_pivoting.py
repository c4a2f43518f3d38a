"""The partial-pivoting items at the edges of their tiles (columns of the padding are
left out, a padded size per 16 / 32 / 64 / 96 / 128): as the choice for every item, and
as the queue of the certified kernels, on a dense vertex whose rho(|M|) exceeds one.

Tolerance: the FP64 path's, max|Delta| / max|ref| <= 1e-12.
"""
import numpy as np
import pytest

from oracle import df_oracle as O
from test_gpu_dense_vertex import dense_problem, rel

pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.mark.parametrize("choice", ["vector", "gjb"])
@pytest.mark.parametrize("n_nu", [2, 8, 10, 16, 18, 32, 34, 40, 48, 50, 56, 58, 64, 66, 80, 82, 96, 98, 112, 114, 128])
def test_pivoting_items(n_nu, choice):
    import torch
    from paper_1507_00895_amd import binding as B
    p, rho_abs = dense_problem(1, 8, n_nu, 1, target=0.9, seed=n_nu)
    x = B.make_instance(p)
    ws = B.workspace([x])
    B.df_autotune_reset()
    B.df_ladder_set_variant(n_nu, B.DF_FP64, choice)
    try:
        B.df_dual_gf([x], ws)
        B.df_bubble([x], ws)
        x.w.fill_(float("nan"))
        B.df_ladder_solve([x], ws)
        torch.cuda.synchronize()
    finally:
        B.df_autotune_reset()
    lr = O.ladder(O.spin_channels(p.gamma_uu, p.gamma_ud), x.chi.cpu().numpy())
    assert choice == "vector" or n_nu < 10 or rho_abs.max() > 1.0
    assert np.array_equal(x.status.cpu().numpy(), lr.status)
    assert rel(x.w.cpu().numpy(), lr.W) <= TOL
    d = x.logdet.cpu().numpy() - lr.logdet
    assert np.abs(np.exp(d) - 1.0).max() <= 1e-10
