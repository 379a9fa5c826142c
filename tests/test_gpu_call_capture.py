"""Kernel-level calls under stream capture: with an MPO tensor that travels in
the launch's arguments a replay gives the captured call's result whatever was
called in between; a larger tensor, whose tables are copied to a buffer that
the next call overwrites, is refused."""
import numpy as np
import pytest

from paper_2005_06104_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_captured_calls_keep_their_tensor_or_are_refused():
    import torch
    from paper_2005_06104_amd import tdvp as T
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        ctx = T.Context(0)
        ml, mr, w = 24, 20, 32
        rng = np.random.default_rng(1)
        dense = [I.random_mpo_site(w, w, k) for k in (2, 3)]
        small = []
        for _ in range(2):
            W = np.zeros(w * w * 4, complex)
            at = rng.permutation(W.size)[:160]
            W[at] = rng.standard_normal(160) + 1j * rng.standard_normal(160)
            small.append(W.reshape(w, w, 2, 2))
        dL, dRt, dC = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (
            I.random_hermitian_env(ml, w, 4), I.random_hermitian_env(mr, w, 5).transpose(1, 2, 0),
            I.random_complex((ml, 2, mr), 6)))
        ws = torch.empty((4 * w + 32) * ml * mr, dtype=torch.complex128, device="cuda")
        Y, Z = torch.empty_like(dC), torch.empty_like(dC)
        T.tdvp_heff_apply(ctx, small[0], dL, dRt, dC, Y, ws)
        ref = Y.clone()
        for _ in range(20):   # every slot of the upload ring has been used
            for W in dense:
                T.tdvp_heff_apply(ctx, W, dL, dRt, dC, Z, ws)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            T.tdvp_heff_apply(ctx, small[0], dL, dRt, dC, Y, ws)
            with pytest.raises(T.TdvpError, match="capture"):
                T.tdvp_heff_apply(ctx, dense[0], dL, dRt, dC, Z, ws)
            with pytest.raises(T.TdvpError, match="capture"):
                T.tdvp_env_right(ctx, dense[0], dRt, dC, torch.empty_like(dL), ws)
        for k in range(4):
            Y.zero_()
            T.tdvp_heff_apply(ctx, (small + dense)[k], dL, dRt, dC, Z, ws)
            g.replay()
            s.synchronize()
            assert torch.equal(Y, ref)
        T.tdvp_heff_apply(ctx, dense[1], dL, dRt, dC, Z, ws)   # the context goes on
        s.synchronize()
        assert bool(torch.isfinite(torch.view_as_real(Z)).all())
        ctx.close()
