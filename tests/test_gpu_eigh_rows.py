"""The reduction with a row of the matrix per wave, at the sizes where its
registers, its gathered columns and its workgroups change, and on values at the
ends of the range; charge blocks that take it next to blocks that do not."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2005_06104_amd import tdvp as T
    ctx = T.Context(0)
    yield T, torch, ctx
    ctx.close()


def _hermitian(n, seed, scale=1.0):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    return scale * (X + X.conj().T)


def _check(lam, V, H):
    n = H.shape[0]
    ref = np.linalg.eigvalsh(H)[::-1]
    s = np.abs(ref).max()
    # the bounds of test_gpu_eigh
    tol = 1e-14 * n + 1e-13
    assert np.abs(lam - ref).max() <= tol * s
    assert np.abs(V @ V.conj().T - np.eye(n)).max() <= tol
    assert np.abs(((V.conj().T * (lam / s)) @ V) - H / s).max() <= tol


@pytest.mark.parametrize("scale", [1.0, 1e-100, 1e100])
@pytest.mark.parametrize("n", [4, 5, 63, 65, 127, 128, 129, 191, 193, 257, 319, 320, 321, 449, 511])
def test_register_and_workgroup_edges(env, n, scale):
    T, torch, ctx = env
    H = _hermitian(n, n, scale)
    dH = torch.from_numpy(H).cuda()
    rows = torch.zeros_like(dH)
    lam = T.tdvp_eigh(ctx, dH, rows, 1)
    _check(lam, rows.cpu().numpy(), H)


@pytest.mark.parametrize("sizes", [(130, 65, 3), (400, 300, 200, 124), (512, 512), (500, 490, 480, 470, 84)])
def test_blocks_of_either_kernel(env, sizes):
    T, torch, ctx = env
    n = sum(sizes)
    q = np.repeat(np.arange(len(sizes)), sizes)
    q = q[np.random.default_rng(n).permutation(n)]
    H = np.where(q[:, None] == q[None, :], _hermitian(n, n), 0.0)
    dH = torch.from_numpy(H).cuda()
    rows = torch.zeros_like(dH)
    lam, qo = T.tdvp_eigh_sectors(ctx, dH, q.astype(np.int32), rows)[:2]
    V = rows.cpu().numpy()
    order = np.argsort(-lam, kind="stable")
    _check(lam[order], V[order], H)
    for i in range(n):   # every row within the block of its charge
        assert np.all(V[i][q != qo[i]] == 0.0)
