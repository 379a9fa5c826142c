"""Products whose operands are read backwards (negative leading dimensions), as
a view of flipped rows is: the same numbers as from a copy in order."""
import pytest

pytestmark = pytest.mark.gpu

# as in test_gpu_gemm_tiles: c bounds a product of the operands' terms, n the
# products per output part and k added up in FP32; FP64 rounds each of the
# 3 K + 64 additions and products of the three real sums, up to 2 |A||B| each
C = {"bf16": 2.0 ** -7 + 2.0 ** -16, "bf16x3": 3.1 * 2.0 ** -16, "fp32": 2.0 ** -24}
N_PRODUCTS = {"bf16": 2, "bf16x3": 6, "fp32": 12}


def _mag(a):
    return a.real.abs() + a.imag.abs()


def _op(a, op):
    return {0: lambda x: x, 1: lambda x: x.mT, 2: lambda x: x.mH, 3: lambda x: x.conj()}[op](a).resolve_conj().contiguous()


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16", "bf16x3"])
@pytest.mark.parametrize("opa,opb", [(0, 0), (1, 2), (2, 3), (3, 1)])
@pytest.mark.parametrize("M,N,K", [(70, 67, 45), (20, 33, 700), (2049, 1023, 65)])
def test_negative_leading_dimensions(prec, opa, opb, M, N, K):
    import torch
    from paper_2005_06104_amd import tdvp as T
    ctx = T.Context(0)
    dt = torch.complex128 if prec == "fp64" else torch.complex64
    g = torch.Generator(device="cuda").manual_seed(M + K)
    rand = lambda *s: torch.randn(*s, dtype=dt, device="cuda", generator=g)  # noqa: E731
    A, B = rand(*((M, K) if opa in (0, 3) else (K, M))), rand(*((K, N) if opb in (0, 3) else (N, K)))
    for fa, fb in ((True, False), (False, True), (True, True)):
        Y = torch.full((M, N), float("nan"), dtype=dt, device="cuda")
        T.tdvp_gemm(ctx, opa, opb, M, N, K, 1.0, A[-1:] if fa else A, -A.shape[1] if fa else A.shape[1], 0,
                    B[-1:] if fb else B, -B.shape[1] if fb else B.shape[1], 0, 0.0, Y, N, 0, 1, prec=prec)
        a, b = (_op((x.flip(0) if f else x).to(torch.complex128), o) for x, f, o in ((A, fa, opa), (B, fb, opb)))
        ref, S = a @ b, _mag(a) @ _mag(b)
        if prec == "fp64":
            bound = 2 * (3 * K + 64) * 2.0 ** -53 * S
        else:
            bound = (C[prec] + (N_PRODUCTS[prec] * K + 64) * 2.0 ** -24) * S + 2.0 ** -22 * ref.abs()
        assert bool(((Y.to(torch.complex128) - ref).abs() <= bound).all())
    ctx.close()
