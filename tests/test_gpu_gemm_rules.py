"""FP64 products on either side of the rules that choose a tile from the blocks a
CU gets (more blocks of one wave than fill its rounds; two narrow tiles a row of
C, dealt in bands or not): right, and the same bits as a few of their rows alone,
which take another tile."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("opa,opb", [(0, 0), (0, 1), (2, 0), (1, 2)])
@pytest.mark.parametrize("M,N,K,batch", [(474, 5086, 50, 1), (474, 4000, 50, 1), (783, 1676, 127, 2), (474, 5086, 33, 2),
                                         (25600, 50, 30, 1), (25601, 50, 30, 1), (2600, 33, 32, 16), (2601, 63, 31, 15)])
def test_rules(opa, opb, M, N, K, batch):
    import torch
    from paper_2005_06104_amd import tdvp as T
    ctx = T.Context(0)
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    rand = lambda *s: torch.randn(*s, dtype=torch.complex128, device="cuda", generator=g)  # noqa: E731
    A, B = rand(batch, *((M, K) if opa == 0 else (K, M))), rand(batch, *((K, N) if opb == 0 else (N, K)))
    op = {0: lambda x: x, 1: lambda x: x.mT, 2: lambda x: x.mH}
    mag = lambda x: x.real.abs() + x.imag.abs()  # noqa: E731
    Y0 = rand(batch, M, N)
    for beta in (0.0, 1.0):
        Y = Y0.clone()
        T.tdvp_gemm(ctx, opa, opb, M, N, K, 1.0, A, A.shape[2], M * K, B, B.shape[2], K * N, beta, Y, N, M * N, batch)
        for b in range(batch):
            a, c = (op[o](x[b]).resolve_conj().contiguous() for x, o in ((A, opa), (B, opb)))
            # as in test_gpu_gemm_beta, here and for the reference
            bound = (4 * (3 * K + 64) * (mag(a) @ mag(c)) + 16 * mag(Y0[b])) * 2.0 ** -53
            assert bool(((Y[b] - (a @ c + beta * Y0[b])).abs() <= bound).all())
        for r in (0, M - 40):
            few = Y0[0, r:r + 40].clone()
            T.tdvp_gemm(ctx, opa, opb, 40, N, K, 1.0, A[0, r:] if opa == 0 else A[0, :, r:], A.shape[2], 0, B, B.shape[2], 0,
                        beta, few, N, 0, 1)
            assert torch.equal(few, Y[0, r:r + 40])
    ctx.close()
