"""Products added to what C holds, on every tile, K part and term image, and on
one short step; rows of C further apart than its columns; the short products
against the staged ones, bit by bit."""
import pytest

pytestmark = pytest.mark.gpu

# as in test_gpu_gemm_tiles: c bounds a product of the operands' terms, n the
# products per output part and k added up in FP32; FP64 rounds each of the
# 3 K + 64 additions and products of the three real sums, up to 2 |A||B| each
C = {"bf16": 2.0 ** -7 + 2.0 ** -16, "bf16x3": 3.1 * 2.0 ** -16, "fp32": 2.0 ** -24}
N_PRODUCTS = {"bf16": 2, "bf16x3": 6, "fp32": 12}


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2005_06104_amd import tdvp as T
    ctx = T.Context(0)
    yield T, torch, ctx
    ctx.close()


def _mag(a):
    return a.real.abs() + a.imag.abs()


def _op(a, op):
    return {0: lambda x: x, 1: lambda x: x.mT, 2: lambda x: x.mH, 3: lambda x: x.conj()}[op](a).resolve_conj().contiguous()


def _operands(torch, dt, opa, opb, M, N, K, batch, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    rand = lambda *s: torch.randn(*s, dtype=dt, device="cuda", generator=g)  # noqa: E731
    return (rand(batch, *((M, K) if opa in (0, 3) else (K, M))), rand(batch, *((K, N) if opb in (0, 3) else (N, K))), rand)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16", "bf16x3"])
@pytest.mark.parametrize("opa,opb", [(0, 0), (1, 2), (3, 1)])
@pytest.mark.parametrize("M,N,K,batch", [(1, 1, 1, 1), (70, 67, 45, 1), (65, 64, 5, 3), (17, 3, 24, 2), (100, 90, 2500, 1),
                                         (300, 33, 257, 1), (2049, 1023, 65, 1), (3000, 2047, 300, 1), (1025, 513, 1500, 1)])
def test_added_to_c(env, prec, opa, opb, M, N, K, batch):
    T, torch, ctx = env
    dt = torch.complex128 if prec == "fp64" else torch.complex64
    A, B, rand = _operands(torch, dt, opa, opb, M, N, K, batch, M + N + K)
    ldc, alpha, beta = N + 3, 0.5 - 2j, -1.5 + 1j
    Y0 = rand(batch, M, ldc)
    Y = Y0.clone()
    T.tdvp_gemm(ctx, opa, opb, M, N, K, alpha, A, A.shape[2], M * K, B, B.shape[2], K * N, beta, Y, ldc, M * ldc, batch,
                prec=prec)
    assert torch.equal(Y[:, :, N:], Y0[:, :, N:])
    for b in range(batch):
        a, c, y0 = (x.to(torch.complex128) for x in (_op(A[b], opa), _op(B[b], opb), Y0[b, :, :N]))
        ref, S = alpha * (a @ c) + beta * y0, 2.5 * (_mag(a) @ _mag(c))
        if prec == "fp64":
            bound = (2 * (3 * K + 64) * S + 16 * _mag(y0)) * 2.0 ** -53
        else:
            bound = (C[prec] + (N_PRODUCTS[prec] * K + 64) * 2.0 ** -24) * S + 2.0 ** -20 * _mag(y0)
        assert bool(((Y[b, :, :N].to(torch.complex128) - ref).abs() <= bound).all())


def test_elements_formed_again_are_added_to_c(env):
    # sums past FP32 on the way (see test_gpu_fp32_again), C of the results' size
    T, torch, ctx = env
    for M, N, K in ((70, 67, 5), (70, 67, 45), (300, 20, 2500)):
        A, B, rand = _operands(torch, torch.complex64, 0, 0, M, N, K, 1, K)
        A, B, Y0 = A[0] * 2.0 ** 50, B[0] * 2.0 ** 54, rand(M, N) * 2.0 ** 104
        # what a product leaves in the scratch of its K parts is not added to the next one's
        T.tdvp_gemm(ctx, 0, 0, M, N, K, 1.0, A * 2.0 ** 12, K, 0, B, N, 0, 0.0, torch.empty_like(Y0), N, 0, 1, prec="fp32")
        Y = Y0.clone()
        T.tdvp_gemm(ctx, 0, 0, M, N, K, 1.0, A, K, 0, B, N, 0, -1.0, Y, N, 0, 1, prec="fp32")
        a, b, y0 = (x.to(torch.complex128) for x in (A, B, Y0))
        bound = 12 * (K + 4) * 2.0 ** -24 * (_mag(a) @ _mag(b)) + 2.0 ** -20 * _mag(y0)
        assert bool(((Y.to(torch.complex128) - (a @ b - y0)).abs() <= bound).all())


@pytest.mark.parametrize("M,N", [(1, 1), (16, 40), (40, 16), (31, 17), (70, 67), (129, 65)])
def test_short_products_are_the_staged_ones(env, M, N):
    # rows of C 2^20 apart take the staged kernel: the same terms and sums
    T, torch, ctx = env
    ld = 1 << 20
    far = torch.empty(M, ld, dtype=torch.complex64, device="cuda")
    for K in (1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 20, 23, 24, 25, 31, 32):
        for opa, opb in ((0, 0), (1, 2), (2, 3), (3, 1)):
            A, B, rand = _operands(torch, torch.complex64, opa, opb, M, N, K, 1, K)
            Y0 = rand(M, N)
            for alpha, beta in ((1.0, 0.0), (0.5 - 2j, 1j)):
                Y, far[:, :N] = Y0.clone(), Y0
                for out, ldc in ((Y, N), (far, ld)):
                    T.tdvp_gemm(ctx, opa, opb, M, N, K, alpha, A, A.shape[2], 0, B, B.shape[2], 0, beta, out, ldc, 0, 1,
                                prec="fp32")
                assert torch.equal(Y, far[:, :N]), (K, opa, opb, beta)


@pytest.mark.parametrize("M,N,batch", [(1000, 1001, 1), (4099, 4900, 1), (21, 2000, 30)])
@pytest.mark.parametrize("K", [3, 16, 17, 24])
def test_large_short_products(env, M, N, batch, K):
    T, torch, ctx = env
    for opa, opb in ((0, 0), (2, 1)):
        A, B, rand = _operands(torch, torch.complex64, opa, opb, M, N, K, batch, K)
        Y = torch.full((batch, M, N), float("nan"), dtype=torch.complex64, device="cuda")
        T.tdvp_gemm(ctx, opa, opb, M, N, K, 1.0, A, A.shape[2], M * K, B, B.shape[2], K * N, 0.0, Y, N, M * N, batch,
                    prec="fp32")
        for b in range(batch):
            a, c = (x.to(torch.complex128) for x in (_op(A[b], opa), _op(B[b], opb)))
            bound = (C["fp32"] + (12 * K + 64) * 2.0 ** -24) * (_mag(a) @ _mag(c))
            assert bool(((Y[b].to(torch.complex128) - a @ c).abs() <= bound).all())
