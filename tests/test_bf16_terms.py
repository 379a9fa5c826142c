"""The three BF16 terms of an FP32 number: exact, and what the six products of
two numbers' terms leave out."""
import numpy as np
import pytest

WORST = np.float32(1 + 2.0 ** -8 - 2.0 ** -17)   # h = 1, m = 2^-8, l = -2^-17


def _bf16(x):
    """nearest BF16 number, ties to even"""
    u = np.asarray(x, dtype=np.float32).view(np.uint32).astype(np.uint64)
    return ((u + 0x7fff + ((u >> 16) & 1)) >> 16 << 16).astype(np.uint32).view(np.float32)


def _terms(x):
    h = _bf16(x)
    m = _bf16(x - h)
    return h, m, x - h - m


def test_terms_hold_the_number_and_leave_less_than_2_to_minus_24():
    rng = np.random.default_rng(3)
    x = np.concatenate([rng.uniform(1, 2, 1 << 20), 1 + np.arange(1 << 12) * 2.0 ** -20, [WORST]]).astype(np.float32)
    h, m, l = _terms(x)
    assert np.array_equal(l, _bf16(l)) and np.array_equal(h.astype(np.float64) + m + l, x.astype(np.float64))
    m, l, x = (np.abs(v).astype(np.float64) for v in (m, l, x))
    # the sums of |m| and |l| that two numbers x, y can bring together
    top = (m / x).max(), (l / x).max()
    assert 2 * top[0] * top[1] + top[1] ** 2 < 2.0 ** -24
    left = (2 * m * l + l * l) / (x * x)
    assert left.max() == left[-1] and 2.0 ** -24.02 < left[-1] < 2.0 ** -24


@pytest.mark.gpu
@pytest.mark.parametrize("M,N", [(1, 1), (70, 67), (6145, 2047)])
def test_worst_products(M, N):
    import torch
    from paper_2005_06104_amd import tdvp as T
    ctx = T.Context(0)
    s = torch.where(torch.arange(M, device="cuda") % 2 == 0, 1.0, -1.0)
    A = (float(WORST) * s).to(torch.complex64).reshape(M, 1).contiguous()
    B = torch.full((1, N), float(WORST), dtype=torch.complex64, device="cuda")
    Y = torch.empty(M, N, dtype=torch.complex64, device="cuda")
    T.tdvp_gemm(ctx, 0, 0, M, N, 1, 1.0, A, 1, 0, B, N, 0, 0.0, Y, N, 0, 1, prec="fp32")
    ref = A.to(torch.complex128) @ B.to(torch.complex128)
    # less than 2^-24 left out, six exact products whose sums round five times
    # (2^-23 each where the matrix cores cut off) and twice outside
    assert bool(((Y.to(torch.complex128) - ref).abs() <= 8 * 2.0 ** -23 * ref.abs()).all())
    ctx.close()
