"""Products at the edges of the tiles and K steps of every tile the dispatch
picks: FP64, and complex64 on the BF16 matrix cores; K splits, conjugations,
leading dimensions past the buffer-addressed range, and operands that have no
BF16 terms (infinities, NaN, numbers that round to an infinity)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# |C - AB| <= (c + (n K + 64) 2^-24) |A||B| in the norm |z| = |Re z| + |Im z|: c
# bounds a product of the operands' terms, n the products per output part and k
# that are added up in FP32 (see test_gpu_kernels; three terms hold an FP32
# number exactly and leave out at most 3 * 2^-26 of a product).
# FP64 rounds each of the 3 K + 64 additions and products of the three real sums
# of a complex product, each sum up to 2 |A||B|.
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


def _operands(torch, opa, opb, M, N, K, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    rand = lambda *s: torch.randn(*s, dtype=torch.complex64, device="cuda", generator=g)  # noqa: E731
    return rand(*((M, K) if opa in (0, 3) else (K, M))), rand(*((K, N) if opb in (0, 3) else (N, K)))


@pytest.mark.parametrize("prec", ["fp32", "bf16", "bf16x3"])
@pytest.mark.parametrize("opa,opb", [(0, 0), (1, 2), (2, 3), (3, 1)])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (16, 15, 8), (63, 65, 31), (64, 64, 32), (65, 63, 33), (129, 127, 97),
                                   (100, 90, 2500), (2049, 1023, 65), (6145, 2047, 40), (1025, 513, 1500)])
def test_tiles_steps_and_splits(env, prec, opa, opb, M, N, K):
    T, torch, ctx = env
    A, B = _operands(torch, opa, opb, M, N, K, 7 * M + N + K)
    Y = torch.full((M, N), float("nan"), dtype=torch.complex64, device="cuda")
    T.tdvp_gemm(ctx, opa, opb, M, N, K, 1.0, A, A.shape[1], 0, B, B.shape[1], 0, 0.0, Y, N, 0, 1, prec=prec)
    a, b = (_op(x.to(torch.complex128), o) for x, o in ((A, opa), (B, opb)))
    ref, S = a @ b, _mag(a) @ _mag(b)
    bound = (C[prec] + (N_PRODUCTS[prec] * K + 64) * 2.0 ** -24) * S + 2.0 ** -22 * ref.abs()
    err = (Y.to(torch.complex128) - ref).abs()
    assert bool((err <= bound).all()), float((err / bound).max())


@pytest.mark.parametrize("opa,opb", [(0, 0), (1, 2), (2, 3), (3, 1)])
@pytest.mark.parametrize("M,N,K,batch", [(1, 1, 1, 1), (16, 15, 5, 1), (17, 33, 127, 1), (64, 32, 256, 1), (97, 95, 193, 2),
                                         (193, 95, 771, 1), (31, 470, 1030, 1), (500, 513, 514, 1), (129, 257, 2050, 1),
                                         (2049, 511, 130, 1), (1100, 1090, 61, 1), (700, 130, 90, 3)])
def test_fp64_tiles_and_parts(env, opa, opb, M, N, K, batch):
    T, torch, ctx = env
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    rand = lambda *s: torch.randn(*s, dtype=torch.complex128, device="cuda", generator=g)  # noqa: E731
    A = rand(batch, *((M, K) if opa in (0, 3) else (K, M)))
    B = rand(batch, *((K, N) if opb in (0, 3) else (N, K)))
    Y0 = rand(batch, M, N)
    Y = Y0.clone()
    T.tdvp_gemm(ctx, opa, opb, M, N, K, 0.5 - 2j, A, A.shape[2], M * K, B, B.shape[2], K * N, -1.0, Y, N, M * N, batch)
    for b in range(batch):
        a, c = _op(A[b], opa), _op(B[b], opb)
        ref = (0.5 - 2j) * (a @ c) - Y0[b]
        bound = (2 * (3 * K + 64) * 2.5 * (_mag(a) @ _mag(c)) + 8 * Y0[b].abs()) * 2.0 ** -53
        assert bool(((Y[b] - ref).abs() <= bound).all())


@pytest.mark.parametrize("opa,opb", [(0, 0), (2, 3)])
def test_fp64_wide_leading_dimension(env, opa, opb):
    # a leading dimension of 2^21 complex128: plain 64-bit addresses
    T, torch, ctx = env
    M, N, K, ld = 40, 33, 37, 1 << 21
    g = torch.Generator(device="cuda").manual_seed(3)
    rand = lambda *s: torch.randn(*s, dtype=torch.complex128, device="cuda", generator=g)  # noqa: E731
    A, B = rand(*((M, K) if opa == 0 else (K, M))), rand(K, N)
    wide = torch.empty(A.shape[0], ld, dtype=torch.complex128, device="cuda")
    wide[:, : A.shape[1]] = A
    Y, Y2 = (torch.empty(M, N, dtype=torch.complex128, device="cuda") for _ in range(2))
    T.tdvp_gemm(ctx, opa, opb, M, N, K, 1.0, wide, ld, 0, B, N, 0, 0.0, Y, N, 0, 1)
    T.tdvp_gemm(ctx, opa, opb, M, N, K, 1.0, A, A.shape[1], 0, B, N, 0, 0.0, Y2, N, 0, 1)
    assert torch.equal(Y, Y2)


@pytest.mark.parametrize("prec", ["fp32", "bf16", "bf16x3"])
@pytest.mark.parametrize("opa,opb", [(0, 0), (1, 1)])
def test_wide_leading_dimension(env, prec, opa, opb):
    # a leading dimension of 2^20 complex64: plain 64-bit addresses
    T, torch, ctx = env
    M, N, K, ld = 70, 33, 37, 1 << 20
    A, B = _operands(torch, opa, opb, M, N, K, 5)
    wide = torch.empty(A.shape[0], ld, dtype=torch.complex64, device="cuda")
    wide[:, : A.shape[1]] = A
    Y = torch.empty(M, N, dtype=torch.complex64, device="cuda")
    Y2 = torch.empty_like(Y)
    T.tdvp_gemm(ctx, opa, opb, M, N, K, 1.0, wide, ld, 0, B, B.shape[1], 0, 0.0, Y, N, 0, 1, prec=prec)
    T.tdvp_gemm(ctx, opa, opb, M, N, K, 1.0, A, A.shape[1], 0, B, B.shape[1], 0, 0.0, Y2, N, 0, 1, prec=prec)
    assert torch.equal(Y, Y2)


@pytest.mark.parametrize("scale", [2.0 ** -100, 2.0 ** -120, 2.0 ** 60, 2.0 ** 100])
def test_fp32_over_the_range_of_its_exponents(env, scale):
    # normal numbers near either end keep their 24 bits (the magnitudes of A
    # reach down to 2^-126 at the smallest scale; at the largest the scaled
    # sums overflow and are formed again)
    T, torch, ctx = env
    M, N, K = 70, 67, 45
    A, B = _operands(torch, 0, 0, M, N, K, 13)
    A = torch.where(_mag(A) < 2.0 ** -4, torch.ones_like(A), A) * scale
    A = torch.complex(torch.where(A.real.abs() < 2.0 ** -126, 0.0, A.real), torch.where(A.imag.abs() < 2.0 ** -126, 0.0, A.imag))
    Y = torch.empty(M, N, dtype=torch.complex64, device="cuda")
    T.tdvp_gemm(ctx, 0, 0, M, N, K, 1.0, A, K, 0, B, N, 0, 0.0, Y, N, 0, 1, prec="fp32")
    a, b = A.to(torch.complex128), B.to(torch.complex128)
    S = _mag(a) @ _mag(b)
    bound = (C["fp32"] + (N_PRODUCTS["fp32"] * K + 64) * 2.0 ** -24) * S
    assert bool(((Y.to(torch.complex128) - a @ b).abs() <= bound).all())


@pytest.mark.parametrize("opa,opb", [(0, 0), (2, 0), (0, 2), (1, 3)])
def test_fp32_operands_without_terms(env, opa, opb):
    # infinities and NaN come out where the three real products of a complex
    # one put them; a finite number that rounds to an infinity in BF16 stays
    # a number
    T, torch, ctx = env
    M, N, K = 70, 67, 45
    A, B = (x.clone() for x in _operands(torch, opa, opb, M, N, K, 11))
    big = 3.4e38
    la, lb = (lambda x, o: x if o in (0, 3) else x.T)(A, opa), (lambda x, o: x if o in (0, 3) else x.T)(B, opb)
    la[3, 5] = complex(float("inf"), 1.0)
    la[64, 44] = complex(1.0, float("-inf"))
    lb[7, 65] = complex(float("nan"), 0.0)
    la[20, :] = 0
    la[20, 9] = complex(big, 0.0)
    lb[9, :] *= 1e-3
    Y = torch.empty(M, N, dtype=torch.complex64, device="cuda")
    T.tdvp_gemm(ctx, opa, opb, M, N, K, 1.0, A, A.shape[1], 0, B, B.shape[1], 0, 0.0, Y, N, 0, 1, prec="fp32")
    a, b = (_op(x.to(torch.complex128), o).cpu().numpy() for x, o in ((A, opa), (B, opb)))
    with np.errstate(invalid="ignore"):
        p1, p2, p3 = a.real @ b.real, a.imag @ b.imag, (a.real + a.imag) @ (b.real + b.imag)
        re, im = p1 - p2, p3 - p1 - p2
        re, im = 1.0 * re - 0.0 * im, 1.0 * im + 0.0 * re      # times alpha = 1 + 0i
    got = Y.cpu().numpy()
    for g, r in ((got.real, re), (got.imag, im)):
        assert np.array_equal(np.isnan(g), np.isnan(r))
        assert np.array_equal(g[np.isinf(r)], r[np.isinf(r)])
        assert np.array_equal(np.isfinite(g), np.isfinite(r))
    S = np.abs(a.real[20]) @ (np.abs(b.real) + np.abs(b.imag))
    fin = np.isfinite(re[20])
    # the 3M form in FP32: every sum rounds on p1, p2, p3, each up to 2 S
    assert (np.abs(got[20] - (re[20] + 1j * im[20]))[fin] <= 12 * (K + 4) * 2.0 ** -24 * S[fin]).all()
