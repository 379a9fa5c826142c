"""Products on term images (one and two BF16 terms): whole, cut into slabs of
rows, of columns and of k, with K splits; partial tiles and k blocks, both
orders of both operands, conjugation, alpha and beta, padded leading
dimensions, operands at 8-byte addresses, infinities."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# see test_gpu_gemm_tiles: c bounds a product of the terms, n the products per
# output part and k that are added up in FP32
C = {"bf16": 2.0 ** -7 + 2.0 ** -16, "bf16x3": 3.1 * 2.0 ** -16}
N_PRODUCTS = {"bf16": 2, "bf16x3": 6}


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


def _padded(torch, g, rows, cols, pad):
    """rows x cols in rows of cols + pad, from an address that is 8 but not 16 bytes aligned"""
    ld = cols + pad
    flat = torch.randn(rows * ld + 1, dtype=torch.complex64, device="cuda", generator=g)[1:]
    return flat, flat.view(rows, ld)[:, :cols], ld


@pytest.mark.parametrize("prec", ["bf16", "bf16x3"])
@pytest.mark.parametrize("opa,opb", [(0, 0), (1, 2), (2, 3), (3, 1)])
@pytest.mark.parametrize("M,N,K", [(1000, 500, 1000), (2049, 1025, 545), (4097, 2049, 1023), (6145, 700, 1021),
                                   (700, 9000, 1021), (1000, 12000, 1023), (12000, 1000, 1023), (1501, 1001, 3500),
                                   (3000, 3000, 3000), (1025, 513, 1500)])
def test_slabs_tiles_and_orders(env, prec, opa, opb, M, N, K):
    T, torch, ctx = env
    g = torch.Generator(device="cuda").manual_seed(M + 3 * N + K)
    fa, A, lda = _padded(torch, g, *((M, K) if opa in (0, 3) else (K, M)), 3)
    fb, B, ldb = _padded(torch, g, *((K, N) if opb in (0, 3) else (N, K)), 0)
    fy, Y, ldy = _padded(torch, g, M, N, 5)
    Y0 = fy.clone().view(M, ldy)
    T.tdvp_gemm(ctx, opa, opb, M, N, K, 0.5 - 2j, fa, lda, 0, fb, ldb, 0, -1.0, fy, ldy, 0, 1, prec=prec)
    a, b = (_op(x.to(torch.complex128), o) for x, o in ((A, opa), (B, opb)))
    ref = (0.5 - 2j) * (a @ b) - Y0[:, :N].to(torch.complex128)
    bound = 2.5 * (C[prec] + (N_PRODUCTS[prec] * K + 64) * 2.0 ** -24) * (_mag(a) @ _mag(b)) + \
        2.0 ** -21 * (ref.abs() + _mag(Y0[:, :N]).double())
    err = (Y.to(torch.complex128) - ref).abs()
    assert bool((err <= bound).all()), float((err / bound).max())
    assert bool((fy.view(M, ldy)[:, N:] == Y0[:, N:]).all())


@pytest.mark.parametrize("prec", ["bf16", "bf16x3"])
def test_special_values_stay_in_their_row_and_column(env, prec):
    T, torch, ctx = env
    M, N, K = 2049, 1025, 545
    g = torch.Generator(device="cuda").manual_seed(5)
    A, B = (torch.randn(*s, dtype=torch.complex64, device="cuda", generator=g) for s in ((M, K), (K, N)))
    A[2048, 544] = complex(np.inf, 1.0)
    B[3, 1024] = complex(np.nan, 0.0)
    Y = torch.zeros((M, N), dtype=torch.complex64, device="cuda")
    T.tdvp_gemm(ctx, 0, 0, M, N, K, 1.0, A, K, 0, B, N, 0, 0.0, Y, N, 0, 1, prec=prec)
    bad = ~(torch.isfinite(Y.real) & torch.isfinite(Y.imag))
    assert bool(bad[2048].all()) and bool(bad[:, 1024].all())
    bad[2048] = False
    bad[:, 1024] = False
    assert not bool(bad.any())
