"""FP32 products with elements that are formed again from the operands (an
infinity, a NaN, sums that the terms' scale takes past FP32): every tile, K
parts and block-sparse items, and at about the speed of other products."""
import numpy as np
import pytest

from paper_2005_06104_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2005_06104_amd import tdvp as T
    ctx = T.Context(0)
    yield T, torch, ctx
    ctx.close()


def _rand(torch, seed, *s):
    return torch.randn(*s, dtype=torch.complex64, device="cuda",
                       generator=torch.Generator(device="cuda").manual_seed(seed))


def _gemm(T, ctx, A, B, Y, opa=0, opb=0):
    (M, K), N = (A.shape if opa in (0, 3) else A.shape[::-1]), B.shape[1 if opb in (0, 3) else 0]
    T.tdvp_gemm(ctx, opa, opb, M, N, K, 1.0, A, A.shape[1], 0, B, B.shape[1], 0, 0.0, Y, N, 0, 1, prec="fp32")


# 128 x 64 tiles; 64 x 64; K parts; a K that ends inside the steps in flight
@pytest.mark.parametrize("opa,opb", [(0, 0), (2, 3), (3, 2), (1, 1)])
@pytest.mark.parametrize("M,N,K,parts", [(6145, 1023, 40, False), (130, 200, 47, False), (100, 90, 2500, True),
                                         (33, 16, 3, False)])
def test_infinities_and_nan(env, opa, opb, M, N, K, parts):
    T, torch, ctx = env
    A = _rand(torch, M, *((M, K) if opa in (0, 3) else (K, M)))
    B = _rand(torch, N, *((K, N) if opb in (0, 3) else (N, K)))
    la, lb = A if opa in (0, 3) else A.T, B if opb in (0, 3) else B.T
    la[M // 2, K // 2] = complex(float("inf"), 1.0)
    la[M - 1, K - 1] = complex(1.0, float("-inf"))
    lb[0, N // 3] = complex(0.5, float("nan"))
    lb[K // 3, N - 1] = complex(float("-inf"), 0.0)
    Y = torch.empty(M, N, dtype=torch.complex64, device="cuda")
    _gemm(T, ctx, A, B, Y, opa, opb)
    a, b = ((x.conj() if o in (2, 3) else x).resolve_conj().cpu().numpy().astype(np.complex128)
            for x, o in ((la, opa), (lb, opb)))
    with np.errstate(invalid="ignore"):
        p1, p2, p3 = a.real @ b.real, a.imag @ b.imag, (a.real + a.imag) @ (b.real + b.imag)
        re, im = p1 - p2, p3 - p1 - p2
        for _ in range(2 if parts else 1):   # times 1 + 0i: the product's, and each K part's
            re, im = 1.0 * re - 0.0 * im, 1.0 * im + 0.0 * re
    got = Y.cpu().numpy()
    for g, r in ((got.real, re), (got.imag, im)):
        assert np.array_equal(np.isnan(g), np.isnan(r))
        assert np.array_equal(g[np.isinf(r)], r[np.isinf(r)])
    fin = np.isfinite(re) & np.isfinite(im)
    a, b = np.where(np.isfinite(a), a, 0), np.where(np.isfinite(b), b, 0)
    S = (np.abs(a.real) + np.abs(a.imag)) @ (np.abs(b.real) + np.abs(b.imag))
    assert (np.abs(got - (re + 1j * im))[fin] <= ((12 * K + 64) * 2.0 ** -24 * S)[fin]).all()


@pytest.mark.parametrize("M,N,K", [(2049, 1023, 65), (100, 90, 2500)])
def test_sums_past_fp32_on_the_way(env, M, N, K):
    # products of 2^104: their sums, times 2^40, are past FP32 and the results
    # are not; the three real sums of the 3M form round K + 4 times each, on up
    # to 2 S
    T, torch, ctx = env
    A, B = _rand(torch, 1, M, K) * 2.0 ** 50, _rand(torch, 2, K, N) * 2.0 ** 54
    Y = torch.empty(M, N, dtype=torch.complex64, device="cuda")
    _gemm(T, ctx, A, B, Y)
    a, b = A.to(torch.complex128), B.to(torch.complex128)
    mag = lambda x: x.real.abs() + x.imag.abs()  # noqa: E731
    assert bool(((Y.to(torch.complex128) - a @ b).abs() <= 12 * (K + 4) * 2.0 ** -24 * (mag(a) @ mag(b))).all())


def test_block_sparse_items(env):
    # the charged matvec is linear in the centre tensor, whose scale takes every
    # sum past FP32 on the way
    from oracle import tdvp as O
    T, torch, ctx = env
    ql, qr = I.charged_bond({-2: 33, 0: 70, 2: 21}), I.charged_bond({-3: 31, -1: 65, 1: 50, 3: 13})
    qwl, qwr = np.array([0, 2, -2, 0, 0], dtype=np.int32), np.array([0, 2, -2, 0], dtype=np.int32)
    rng = np.random.default_rng(7)
    ps = np.array([1, -1])
    W = rng.standard_normal((5, 4, 2, 2)) + 1j * rng.standard_normal((5, 4, 2, 2))
    W[ps[None, None, None, :] - qwl[:, None, None, None] != ps[None, None, :, None] - qwr[None, :, None, None]] = 0
    L, R, C = (x.astype(np.complex64).astype(np.complex128) for x in I.random_charged_heff_operands(ql, qr, qwl, qwr, 9))
    scale = 2.0 ** 100
    dL, dRt, dC = (torch.from_numpy(np.ascontiguousarray(x)).to(torch.complex64).cuda()
                   for x in (L, R.transpose(1, 2, 0), C * scale))
    dY = torch.full(C.shape, float("nan"), dtype=torch.complex64, device="cuda")
    T.tdvp_heff_apply_u1(ctx, W, dL, dRt, dC, dY, ql, qr, qwl, qwr)
    Y = dY.cpu().numpy().astype(np.complex128) / scale
    # two products of at most max(K) complex terms (three sums each) around the
    # stage, on the magnitudes |Re z| + |Im z|
    mag = lambda a: (np.abs(a.real) + np.abs(a.imag)).astype(np.complex128)  # noqa: E731
    S = O.heff_apply(mag(L), mag(W), mag(R), mag(C)).real
    K = max(L.shape[2], R.shape[1] * R.shape[2])
    assert (np.abs(Y - O.heff_apply(L, W, R, C)) <= 8 * (3 * K + 64) * 2.0 ** -24 * S).all()
    allowed = qr[None, None, :] == ql[:, None, None] + ps[None, :, None]
    assert np.all(Y[~allowed] == 0)


@pytest.mark.parametrize("what", ["sums", "nan"])
def test_at_about_the_speed_of_other_products(env, what):
    # the elements' second sums take the FP32 matrix cores about twice the time
    # of the first; one lane an element took 30 to 50 times the whole product
    T, torch, ctx = env
    M, N, K = 2048, 2048, 1024
    A, B = _rand(torch, 1, M, K), _rand(torch, 2, K, N)
    A2 = A * 2.0 ** 100 if what == "sums" else A.clone()
    if what == "nan":
        A2[:, 7] = float("nan")
    Y = torch.empty(M, N, dtype=torch.complex64, device="cuda")

    def best(a):
        t = []
        for _ in range(6):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            _gemm(T, ctx, a, B, Y)
            e[1].record()
            e[1].synchronize()
            t.append(e[0].elapsed_time(e[1]))
        return min(t)
    assert best(A2) <= 8 * best(A)
