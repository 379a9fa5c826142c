"""Matrices that are not finite end in TDVP_ERR_NUMERIC, through the own solver
alone and through the automatic choice, dense and in charge blocks, and the
next decomposition is right; very small numbers are scaled without an
infinite inverse."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _hermitian(n, seed):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    return X + X.conj().T


def _check(lam, V, H):
    n = H.shape[0]
    tol = 1e-14 * n + 1e-13      # the bounds of test_gpu_eigh
    ref = np.linalg.eigvalsh(H)[::-1]
    s = np.abs(ref).max()
    assert np.abs(lam - ref).max() <= tol * s
    assert np.abs(V @ V.conj().T - np.eye(n)).max() <= tol


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("n", [2, 16, 17, 40, 128, 300, 512])
def test_non_finite_matrices_are_an_error(n, value):
    import torch
    from paper_2005_06104_amd import tdvp as T
    ctx = T.Context(0)
    good = _hermitian(n, n)
    for at in ((0, 0), (n // 2, n // 2), (n - 1, 0)):
        H = good.copy()
        H[at] = H[at[::-1]] = value
        dH = torch.from_numpy(H).cuda()
        rows = torch.zeros_like(dH)
        for method in (1, 0):
            with pytest.raises(T.TdvpError) as e:
                T.tdvp_eigh(ctx, dH, rows, method)
            assert e.value.status == T.TDVP_ERR_NUMERIC
        q = np.arange(n, dtype=np.int32) % 2       # two blocks, side by side
        if n >= 4 and at[0] % 2 == at[1] % 2:
            with pytest.raises(T.TdvpError) as e:
                T.tdvp_eigh_sectors(ctx, torch.where(torch.from_numpy(q[:, None] == q[None, :]).cuda(), dH, 0.0), q, rows)
            assert e.value.status == T.TDVP_ERR_NUMERIC
        dG = torch.from_numpy(good).cuda()
        _check(T.tdvp_eigh(ctx, dG, rows, 1), rows.cpu().numpy(), good)
    ctx.close()


def test_diagonals_down_to_the_smallest_numbers():
    import torch
    from paper_2005_06104_amd import tdvp as T
    ctx = T.Context(0)
    n = 40
    d = np.arange(n) * 5e-324
    dH = torch.from_numpy(np.diag(d).astype(complex)).cuda()
    rows = torch.zeros_like(dH)
    lam = T.tdvp_eigh(ctx, dH, rows, 1)
    assert np.array_equal(lam, d[::-1])
    V = rows.cpu().numpy()
    assert np.abs(V @ V.conj().T - np.eye(n)).max() == 0.0
    ctx.close()
