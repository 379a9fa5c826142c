"""MPO tensors at the limits of what travels with a launch (160 nonzeros, 64
output channels) and one past them, rows without entries and an empty tensor,
in every precision."""
import numpy as np
import pytest

from paper_2005_06104_amd import inputs as I

pytestmark = pytest.mark.gpu

# rounding of the sums in FP64, of three BF16 terms and FP32 sums, of two terms
TOL = {"fp64": 1e-12, "fp32": 2e-5, "bf16x3": 1e-3}


@pytest.mark.parametrize("prec", sorted(TOL))
@pytest.mark.parametrize("wl,wr,nnz", [(32, 32, 160), (32, 32, 161), (31, 32, 1), (32, 1, 64), (1, 32, 128), (8, 5, 160),
                                       (3, 4, 0)])
def test_inline_limits(prec, wl, wr, nnz):
    import torch
    from oracle import tdvp as O
    from paper_2005_06104_amd import tdvp as T
    ctx = T.Context(0)
    ml, mr = 21, 34
    rng = np.random.default_rng(nnz + wl)
    W = np.zeros(wl * wr * 4, complex)
    at = rng.permutation(W.size)[:nnz]
    W[at] = rng.standard_normal(nnz) + 1j * rng.standard_normal(nnz)
    W = W.reshape(wl, wr, 2, 2)
    L, R = I.random_hermitian_env(ml, wl, 1), I.random_hermitian_env(mr, wr, 2)
    C = I.random_complex((ml, 2, mr), 3)
    dt = torch.complex128 if prec == "fp64" else torch.complex64
    dL, dRt, dC = (torch.from_numpy(np.ascontiguousarray(x)).to(dt).cuda() for x in (L, R.transpose(1, 2, 0), C))
    Y = torch.full_like(dC, float("nan"))
    E = torch.full((wl, ml, ml), float("nan"), dtype=dt, device="cuda")
    ws = torch.empty((4 * max(wl, wr) + 32) * ml * mr, dtype=dt, device="cuda")
    p = prec if prec == "bf16x3" else None
    T.tdvp_heff_apply(ctx, W, dL, dRt, dC, Y, ws, prec=p)
    T.tdvp_env_right(ctx, W, dRt, dC, E, ws, prec=p)
    torch.cuda.synchronize()
    ref, refE = O.heff_apply(L, W, R, C), O.right_env_update(R, C, W).transpose(1, 2, 0)
    for got, want in ((Y, ref), (E, refE)):
        assert np.abs(got.cpu().numpy() - want).max() <= TOL[prec] * np.abs(want).max()
    ctx.close()
