"""Kernel-level calls with a workspace: asynchronous for a caller on the context's
stream; one on another stream finds the result there, and may drop its tensors,
when the call returns."""
import numpy as np
import pytest

from paper_2005_06104_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_caller_on_another_stream(prec):
    import torch
    from paper_2005_06104_amd import tdvp as T
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        ctx = T.Context(0)
    ml, mr, w = 600, 500, 12
    dt = torch.complex128 if prec == "fp64" else torch.complex64
    dL, dRt, dC = (torch.from_numpy(np.ascontiguousarray(x)).to(dt).cuda() for x in (
        I.random_hermitian_env(ml, w, 4), I.random_hermitian_env(mr, w, 5).transpose(1, 2, 0),
        I.random_complex((ml, 2, mr), 6)))
    W = I.random_mpo_site(w, w, 2)
    ws = torch.empty((4 * w + 32) * ml * mr, dtype=dt, device="cuda")
    Lout = torch.empty(mr, w, mr, dtype=dt, device="cuda")
    Rout = torch.empty(w, ml, ml, dtype=dt, device="cuda")
    calls = (lambda y: T.tdvp_heff_apply(ctx, W, dL, dRt, dC, y, ws), lambda y: T.tdvp_env_left(ctx, W, dL, dC, y, ws),
             lambda y: T.tdvp_env_right(ctx, W, dRt, dC, y, ws))
    for call, out in zip(calls, (dC, Lout, Rout)):
        ref, Y = torch.empty_like(out), torch.empty_like(out)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            call(ref)
        torch.cuda.synchronize()
        call(Y)
        assert side.query()
        assert torch.equal(Y, ref)
    ctx.close()
