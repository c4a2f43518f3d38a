"""Non-finite vertex elements, at positions in different lanes, waves and work-groups of
the symmetry check: the ladders of that bosonic index and channel are non-finite (status
2), the others are untouched, and df_lattice hands the value on."""
import numpy as np
import pytest

from paper_1507_00895_amd import inputs as I

pytestmark = pytest.mark.gpu


def solve(p):
    import torch
    from paper_1507_00895_amd import binding as B
    inst = B.make_instance(p)
    ws = B.workspace([inst])
    B.df_dual_gf([inst], ws)
    B.df_bubble([inst], ws)
    B.df_ladder_solve([inst], ws)
    torch.cuda.synchronize()
    return inst.status.cpu().numpy(), inst.w.cpu().numpy()


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("n_nu,i,j", [(14, 0, 0), (14, 0, 5), (48, 0, 17), (48, 5, 15), (48, 47, 46),
                                      (64, 3, 62), (64, 63, 63), (128, 70, 1)])
def test_a_nonfinite_vertex_element(n_nu, i, j, value):
    import torch
    from paper_1507_00895_amd import binding as B
    p = I.atomic_limit_problem(2, 8, n_nu, 3, 10.0, 2.0, 0.1)
    ok_st, ok_w = solve(p)
    assert (ok_st == 0).all()
    p.gamma_uu = p.gamma_uu.copy()
    p.gamma_uu[1, i, j] = p.gamma_uu[1, j, i] = value
    st, w = solve(p)
    assert (st[:, 1] == 2).all()
    assert np.array_equal(st[:, [0, 2]], ok_st[:, [0, 2]])
    assert np.array_equal(w[:, [0, 2]], ok_w[:, [0, 2]])
    x = B.make_instance(p, outputs=False)
    ch, sp = (torch.empty(p.N, dtype=torch.complex128, device="cuda") for _ in range(2))
    B.df_lattice(x, p.mu, None, None, ch, sp)
    torch.cuda.synchronize()
    assert not np.isfinite(ch.cpu().numpy()).any() and not np.isfinite(sp.cpu().numpy()).any()
