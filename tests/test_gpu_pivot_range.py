"""Partial pivoting where the pivots are far from one: |1 - gamma chi| up to 1e+-170 (chi in
units of its own, gamma in the inverse ones are both legitimate; the matrix need not be
near one where the ladder diverges).  log det and status against the oracle; 1e-11, the
FP64 path's."""
import numpy as np
import pytest

from oracle import df_oracle as O
from paper_1507_00895_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel", ["gjb", "vector"])
@pytest.mark.parametrize("n_nu,nk", [(14, 8), (48, 8), (64, 32), (80, 8), (128, 8)])
def test_large_pivots(n_nu, nk, kernel):
    import torch
    from paper_1507_00895_amd import binding as B
    p = I.atomic_limit_problem(2, nk, n_nu, 1, 10.0, 2.0, 0.1)
    rng = np.random.default_rng(n_nu)
    z = lambda s: rng.standard_normal(s) + 1j * rng.standard_normal(s)
    p.gamma_uu, p.gamma_ud = z((1, n_nu, n_nu)), z((1, n_nu, n_nu))
    chi = 1e170 * z((1, n_nu, p.N))
    inst = B.make_instance(p)
    inst.chi.copy_(torch.as_tensor(chi))
    B.df_ladder_set_variant(n_nu, B.DF_FP64, kernel)
    try:
        B.df_ladder_solve([inst], B.workspace([inst]))
        torch.cuda.synchronize()
    finally:
        B.df_autotune_reset()
    pick = rng.integers(0, p.N, 16)
    ref = O.ladder(O.spin_channels(p.gamma_uu, p.gamma_ud), chi[:, :, pick])
    st, ld = inst.status.cpu().numpy()[..., pick], inst.logdet.cpu().numpy()[..., pick]
    assert np.array_equal(st, ref.status)
    # (log |det| is about n_nu * 391)
    assert np.abs(ld.real / ref.logdet.real - 1).max() <= 1e-11
    assert np.abs(np.exp(1j * ld.imag) - np.exp(1j * ref.logdet.imag)).max() <= 1e-11
    w = inst.w.cpu().numpy()[..., pick]
    assert np.abs(w - ref.W).max() <= 1e-12 * np.abs(ref.W).max()
