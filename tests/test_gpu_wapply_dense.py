"""The sparse-MPO stage of large operands through LDS: tensors with many
nonzeros, ragged columns, charges that change inside a block of columns."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

PS = np.array([1, -1])


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2005_06104_amd import tdvp as T
    ctx = T.Context(0)
    yield T, torch, ctx
    ctx.close()


def _heff(torch, L, W, Rt, C):
    ml, wl, _ = L.shape
    wr, mr, _ = Rt.shape
    t = (L.reshape(ml * wl, ml) @ C.reshape(ml, 2 * mr)).reshape(ml, wl, 2, mr).permute(0, 3, 1, 2).reshape(ml * mr, 2 * wl)
    t = t.contiguous() @ W.permute(0, 3, 1, 2).reshape(2 * wl, 2 * wr).contiguous()     # (al, s) -> (be, s')
    t = t.reshape(ml, mr, wr, 2).permute(0, 3, 2, 1).reshape(2 * ml, wr * mr).contiguous()
    return (t @ Rt.reshape(wr * mr, mr)).reshape(ml, 2, mr)


def _check(torch, prec, got, L, W, Rt, C):
    mag = lambda a: (a.real.abs() + a.imag.abs()).to(torch.complex128)  # noqa: E731
    ref, S = _heff(torch, L, W, Rt, C), _heff(torch, mag(L), mag(W), mag(Rt), mag(C)).real
    # two products of at most max(K) complex terms (three sums each) around a
    # stage of at most 64, on the magnitudes |Re z| + |Im z|
    K = max(L.shape[2], Rt.shape[0] * Rt.shape[1])
    u = 2.0 ** -53 if prec == "fp64" else 2.0 ** -24
    assert bool(((got.to(torch.complex128) - ref).abs() <= 8 * (3 * K + 64 + 4 * 64) * u * S).all())


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("ml,wl,wr,mr,share", [(1400, 5, 4, 130, 1.0), (512, 32, 32, 511, 0.4), (1366, 17, 32, 129, 0.9),
                                               (1365, 17, 3, 129, 0.9), (4100, 4, 6, 1, 1.0)])
def test_many_nonzeros(env, prec, ml, wl, wr, mr, share):
    T, torch, ctx = env
    dt = torch.complex128 if prec == "fp64" else torch.complex64
    g = torch.Generator(device="cuda").manual_seed(ml)
    L, Rt, C = (torch.randn(*s, dtype=dt, device="cuda", generator=g) for s in ((ml, wl, ml), (wr, mr, mr), (ml, 2, mr)))
    rng = np.random.default_rng(wl)
    W = rng.standard_normal((wl, wr, 2, 2)) + 1j * rng.standard_normal((wl, wr, 2, 2))
    W[rng.random(W.shape) >= share] = 0
    Y = torch.full((ml, 2, mr), float("nan"), dtype=dt, device="cuda")
    T.tdvp_heff_apply(ctx, W, L, Rt, C, Y, prec=prec)
    c128 = lambda x: x.to(torch.complex128)  # noqa: E731
    _check(torch, prec, Y, c128(L), torch.from_numpy(W).cuda(), c128(Rt), c128(C))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_many_nonzeros_with_charges(env, prec):
    T, torch, ctx = env
    dt = torch.complex128 if prec == "fp64" else torch.complex64
    ml, w, cut, mr = 1400, 32, 67, 131
    ql = np.zeros(ml, dtype=np.int32)
    qr = np.where(np.arange(mr) < cut, -1, 1).astype(np.int32)
    qw = np.zeros(w, dtype=np.int32)
    g = torch.Generator(device="cuda").manual_seed(4)
    L, Rt, C = (torch.randn(*s, dtype=dt, device="cuda", generator=g) for s in ((ml, w, ml), (w, mr, mr), (ml, 2, mr)))
    Rt[:, :cut, cut:] = 0
    Rt[:, cut:, :cut] = 0
    C[:, 0, :cut] = 0
    C[:, 1, cut:] = 0
    rng = np.random.default_rng(2)
    W = rng.standard_normal((w, w, 2, 2)) + 1j * rng.standard_normal((w, w, 2, 2))
    W[:, :, 0, 1] = W[:, :, 1, 0] = 0
    Y = torch.full((ml, 2, mr), float("nan"), dtype=dt, device="cuda")
    T.tdvp_heff_apply_u1(ctx, W, L, Rt, C, Y, ql, qr, qw, qw, prec=prec)
    c128 = lambda x: x.to(torch.complex128)  # noqa: E731
    _check(torch, prec, Y, c128(L), torch.from_numpy(W).cuda(), c128(Rt), c128(C))
    assert bool((Y[:, 0, :cut] == 0).all()) and bool((Y[:, 1, cut:] == 0).all())
