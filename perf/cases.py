"""Timed cases of the GSE-TDVP1 library: what its users call, over the sizes
their runs go through.

A time step spends its time in the one-site effective Hamiltonian (the matvec
of the local Lanczos runs), the zero-site one, the environment updates, and
the FP64 factorisations of the gauge moves and truncations; each has a case
through its own entry point, and one case is a whole sweep with its
measurement.  Sizes follow the workloads of ``inputs.py``: the 2x6 ladder
(bonds up to 32), the 2x32 ladder (256, FP64), the 2x64 ladder (512, FP32) and
the 4x16 J1-J2 cylinder (1024, MPO bonds 14 to 20, dense and with U(1)
charges); bond dimensions after a truncation are whatever the cut leaves, so
odd ones are as common as round ones.

Operands have the magnitudes the method gives them: the finished channel of an
environment is the identity, the others are O(1) operators, a centre tensor
has a decaying Schmidt spectrum, the MPO tensor is a sparse automaton of
S^+, S^-, S^z channels.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2005_06104_amd import tdvp as T

# share of the states of a cylinder's middle bonds in each S^z sector
EVEN_SECTORS = {-4: 0.078, -2: 0.281, 0: 0.381, 2: 0.238, 4: 0.022}
ODD_SECTORS = {-5: 0.029, -3: 0.176, -1: 0.322, 1: 0.313, 3: 0.146, 5: 0.014}

OPS = {"N": T.OP_N, "T": T.OP_T, "C": T.OP_C, "R": T.OP_R}


def listed():
    return [
        # the 2x6 ladder's matvec: four small launches, latency counts
        dict(name="heff_fp64_c32", kind="heff", prec="fp64", ml=32, mr=32, wl=8, wr=8),
        # the 2x32 ladder at its bond cap, the FP64 headline size
        dict(name="heff_fp64_c256", kind="heff", prec="fp64", ml=256, mr=256, wl=8, wr=8),
        # the 2x64 ladder near its cap, in FP32, bonds as a cut leaves them
        dict(name="heff_fp32_c500", kind="heff", prec="fp32", ml=487, mr=512, wl=8, wr=8),
        # the cylinder's matvec without symmetry: the largest products
        dict(name="heff_fp32_c1024", kind="heff", prec="fp32", ml=1024, mr=1024, wl=20, wr=20),
        # the cylinder's matvec with its S^z charges
        dict(name="heff_u1_fp32_c1024", kind="heff_u1", prec="fp32", ml=1024, mr=1009, wl=17, wr=20),
        # left environment update in the split BF16 precision
        dict(name="env_left_bf16x3_c768", kind="env_left", prec="bf16x3", ml=768, mr=701, wl=14, wr=17),
        # right environment update of the FP64 ladder, ragged bonds
        dict(name="env_right_fp64_c231", kind="env_right", prec="fp64", ml=231, mr=256, wl=8, wr=8),
        # zero-site matvec of the 2x64 ladder
        dict(name="keff_fp32_c512", kind="keff", prec="fp32", ml=512, mr=509, wl=8, wr=8),
        # one product in plain BF16, a cylinder's L . C
        dict(name="gemm_bf16", kind="gemm", prec="bf16", opa="N", opb="N", m=14000, n=2048, k=1021, batch=1),
        # Cholesky factor and inverse of a gauge move's Gram matrix
        dict(name="cholesky_n300", kind="cholesky", n=300),
        # eigendecomposition of a density matrix of the 2x32 ladder
        dict(name="eigh_n512", kind="eigh", n=512),
        # a whole FP64 sweep of a 2x10 ladder and the measurement after it
        dict(name="sweep_fp64_c96", kind="sweep", legs=10, chi=96, dt=0.05),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["heff", "heff", "heff_u1", "env_left", "env_right", "keff", "gemm", "cholesky", "eigh", "sweep"])
    if kind in ("heff", "env_left", "env_right", "keff"):
        prec = rng.choice(["fp64", "fp32", "bf16x3"])
        ml = _log(rng, 16, 320) if prec == "fp64" else _log(rng, 48, 1000)
        mr = max(8, min(2 * ml, int(ml * rng.uniform(0.7, 1.4)), 320 if prec == "fp64" else 1000))
        wl = rng.randint(5, 20)
        wr = max(5, min(20, wl + rng.randint(-3, 3))) if kind != "keff" else wl
        return dict(kind=kind, prec=prec, ml=ml, mr=mr, wl=wl, wr=wr)
    if kind == "heff_u1":
        wl = rng.randint(8, 20)
        return dict(kind=kind, prec=rng.choice(["fp64", "fp32", "bf16x3"]), ml=_log(rng, 200, 1000),
                    mr=_log(rng, 200, 1000), wl=wl, wr=max(8, min(20, wl + rng.randint(-3, 3))))
    if kind == "gemm":
        prec = rng.choice(["fp64", "fp32", "bf16", "bf16x3"])
        top = 1200 if prec == "fp64" else 3000
        return dict(kind=kind, prec=prec, opa=rng.choice("NTCR"), opb=rng.choice("NTCR"), m=_log(rng, 16, top),
                    n=_log(rng, 16, top), k=_log(rng, 16, top), batch=rng.choice([1, 1, 2, 5]))
    if kind in ("cholesky", "eigh"):
        return dict(kind=kind, n=_log(rng, 12, 512))
    return dict(kind=kind, legs=rng.randint(4, 10), chi=_log(rng, 12, 96), dt=round(rng.uniform(0.02, 0.1), 3))


# ------------------------------------------------------------------ inputs
@functools.lru_cache(maxsize=None)
def _context():
    return T.Context(torch.cuda.current_device())


def _gauss(gen, *shape):
    return torch.randn(*shape, dtype=torch.complex128, device="cuda", generator=gen)


def _dtype(case):
    return torch.complex128 if case["prec"] == "fp64" else torch.complex64


def mpo_site(wl, wr, seed):
    """W[alpha, beta, s', s] of a Heisenberg-type automaton, with the S^z
    charges of its channels: channel 0 has not started, the last has finished,
    those between carry S^+, S^-, S^z in turn; three open here, three close
    here, the others pass."""
    rng = np.random.default_rng(seed)
    sp, sm, sz = np.array([[0, 1], [0, 0]]), np.array([[0, 0], [1, 0]]), np.array([[0.5, 0], [0, -0.5]])
    start, close = [sp, sm, sz], [sm, sp, sz]
    w = np.zeros((wl, wr, 2, 2), dtype=np.complex128)
    w[0, 0] = w[-1, -1] = np.eye(2)
    for c in range(1, min(wl, wr) - 1):
        w[c, c] = np.eye(2)
    for c in range(max(1, wr - 4), wr - 1):
        w[0, c] = start[(c - 1) % 3]
        if c < wl - 1:
            w[c, c] = 0
    for c in range(1, min(4, wl - 1)):
        w[c, -1] = rng.uniform(0.5, 1.5) * close[(c - 1) % 3]
    w[0, -1] = rng.uniform(-0.5, 0.5) * sz
    q = lambda n: np.array([0] + [(2, -2, 0)[(c - 1) % 3] for c in range(1, n - 1)] + [0], dtype=np.int32)  # noqa: E731
    return w, q(wl), q(wr)


def charges(m, sectors):
    sizes = {c: max(1, int(f * m)) for c, f in sectors.items()}
    biggest = max(sizes, key=sizes.get)
    sizes[biggest] += m - sum(sizes.values())
    return np.repeat(np.array(sorted(sizes), dtype=np.int32), [sizes[c] for c in sorted(sizes)])


def _environment(gen, m, w, bra_last):
    """(m, w, m) as [a', alpha, a], or (w, m, m) as [beta, b, b']"""
    e = _gauss(gen, m, w, m) / math.sqrt(m)
    first = -1 if bra_last else 0
    e[:, first, :] = torch.eye(m, dtype=e.dtype, device=e.device)
    return e.permute(1, 2, 0).contiguous() if bra_last else e


def _decay(m, q=None):
    pos = torch.arange(m, dtype=torch.float64, device="cuda") / m
    if q is not None:      # each sector has its own spectrum
        pos = torch.cat([torch.arange(n, dtype=torch.float64) / n for n in np.unique(q, return_counts=True)[1]]).cuda()
    return 10.0 ** (-3.0 * pos)


def _operands(case, seed):
    """Operands of the contraction cases in the case's precision, W on the host."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    ml, mr, wl, wr = (case[k] for k in ("ml", "mr", "wl", "wr"))
    W, qwl, qwr = mpo_site(wl, wr, seed)
    o = dict(W=W, qwl=qwl, qwr=qwr, ql=None, qr=None)
    kind = case["kind"]
    if kind != "env_right":
        o["L"] = _environment(gen, ml, wl, False)
    if kind != "env_left":
        o["Rt"] = _environment(gen, mr, wr, True)
    if kind == "keff":
        x = _gauss(gen, ml, mr) * _decay(ml)[:, None] * _decay(mr)[None, :]
        o["C"] = x / torch.linalg.vector_norm(x)
    elif kind in ("env_left", "env_right"):   # an isometry up to rounding of its Gram matrix
        o["C"] = _gauss(gen, ml, 2, mr) / math.sqrt(2 * (ml if kind == "env_left" else mr))
    else:
        ql = charges(ml, EVEN_SECTORS) if kind == "heff_u1" else None
        qr = charges(mr, ODD_SECTORS) if kind == "heff_u1" else None
        x = _gauss(gen, ml, 2, mr) * _decay(ml, ql)[:, None, None] * _decay(mr, qr)[None, None, :]
        if kind == "heff_u1":
            o["ql"], o["qr"] = ql, qr
            a, b, ca, cb = (torch.from_numpy(v).cuda() for v in (ql, qr, qwl, qwr))
            o["L"] *= a[None, None, :] == a[:, None, None] - ca[None, :, None]
            o["Rt"] *= b[None, :, None] == b[None, None, :] - cb[:, None, None]
            s = torch.tensor([1, -1], device="cuda")
            x *= b[None, None, :] == a[:, None, None] + s[None, :, None]
        o["C"] = x / torch.linalg.vector_norm(x)
    for k in ("L", "Rt", "C"):
        if k in o:
            o[k] = o[k].to(_dtype(case))
    return o


def _gemm_operands(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    m, n, k, b = (case[x] for x in ("m", "n", "k", "batch"))
    A = _gauss(gen, b, *((m, k) if case["opa"] in "NR" else (k, m))).to(_dtype(case))
    B = _gauss(gen, b, *((k, n) if case["opb"] in "NR" else (n, k))).to(_dtype(case))
    return A, B


def _gram(case, seed):
    """A Gram matrix as gauge moves and density matrices have it, weights falling off"""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    n = case["n"]
    x = _gauss(gen, 2 * n, n) * 10.0 ** (-torch.arange(n, device="cuda", dtype=torch.float64) / n)
    g = x.mH @ x
    return (0.5 * (g + g.mH) / torch.linalg.matrix_norm(x) ** 2).contiguous()


def ladder_couplings(legs):
    """Two-leg Heisenberg ladder on the snake path: (i, j) with J = 1"""
    at = lambda x, r: 2 * x + (r if x % 2 == 0 else 1 - r)  # noqa: E731
    bonds = [(at(x, r), at(x + 1, r)) for x in range(legs - 1) for r in (0, 1)] + [(at(x, 0), at(x, 1)) for x in range(legs)]
    return sorted((min(b), max(b)) for b in bonds)


def _chain_state(case, seed):
    """A random normalised MPS in right-canonical form, the centre on site 0"""
    rng = np.random.default_rng(seed)
    n = 2 * case["legs"]
    dims = [min(case["chi"], 2 ** min(i, n - i)) for i in range(n + 1)]
    t = [rng.standard_normal((dims[i], 2, dims[i + 1])) + 1j * rng.standard_normal((dims[i], 2, dims[i + 1])) for i in range(n)]
    for i in range(n - 1, 0, -1):
        q, r = np.linalg.qr(t[i].reshape(dims[i], -1).conj().T)
        t[i] = q.conj().T.reshape(dims[i], 2, dims[i + 1])
        t[i - 1] = np.tensordot(t[i - 1], r.conj().T, 1)
    t[0] /= np.linalg.norm(t[0])
    return t


# --------------------------------------------------------------- the cases
def prepare(case, seed):
    ctx, kind = _context(), case["kind"]
    s = dict(kind=kind, case=case, ctx=ctx)
    if kind == "gemm":
        s["A"], s["B"] = _gemm_operands(case, seed)
        s["Y"] = torch.zeros(case["batch"], case["m"], case["n"], dtype=_dtype(case), device="cuda")
    elif kind == "cholesky":
        s["G"] = _gram(case, seed)
        s["L"], s["Linv"] = torch.zeros_like(s["G"]), torch.zeros_like(s["G"])
    elif kind == "eigh":
        s["G"] = _gram(case, seed)
        s["rows"] = torch.zeros_like(s["G"])
    elif kind == "sweep":
        n = 2 * case["legs"]
        terms = [(i, j, a, b, c) for i, j in ladder_couplings(case["legs"]) for a, b, c in ((3, 3, 1.0), (1, 2, 0.5), (2, 1, 0.5))]
        s["H"] = T.tdvp_create_mpo(ctx, n, terms)
        s["psi"] = T.tdvp_mps_from_host(ctx, _chain_state(case, seed))
    else:
        s.update(_operands(case, seed))
        ml, mr, wl, wr = (case[k] for k in ("ml", "mr", "wl", "wr"))
        shape = {"env_left": (mr, wr, mr), "env_right": (wl, ml, ml), "keff": (ml, mr)}.get(kind, (ml, 2, mr))
        s["Y"] = torch.zeros(shape, dtype=_dtype(case), device="cuda")
        s["prec"] = case["prec"] if case["prec"].startswith("bf16") else None
        if kind != "heff_u1":   # kept by a program that applies the operator many times
            s["work"] = torch.empty((4 * max(wl, wr) + 32) * ml * mr, dtype=_dtype(case), device="cuda")
    return s


def run(s):
    ctx, kind, case = s["ctx"], s["kind"], s["case"]
    if kind == "heff":
        T.tdvp_heff_apply(ctx, s["W"], s["L"], s["Rt"], s["C"], s["Y"], s["work"], prec=s["prec"])
    elif kind == "heff_u1":
        T.tdvp_heff_apply_u1(ctx, s["W"], s["L"], s["Rt"], s["C"], s["Y"], s["ql"], s["qr"], s["qwl"], s["qwr"],
                             prec=s["prec"])
    elif kind == "keff":
        T.tdvp_keff_apply(ctx, s["L"], s["Rt"], s["C"], s["Y"], s["work"], prec=s["prec"])
    elif kind == "env_left":
        T.tdvp_env_left(ctx, s["W"], s["L"], s["C"], s["Y"], s["work"], prec=s["prec"])
    elif kind == "env_right":
        T.tdvp_env_right(ctx, s["W"], s["Rt"], s["C"], s["Y"], s["work"], prec=s["prec"])
    elif kind == "gemm":
        A, B, Y = s["A"], s["B"], s["Y"]
        T.tdvp_gemm(ctx, OPS[case["opa"]], OPS[case["opb"]], case["m"], case["n"], case["k"], 1.0, A, A.shape[2],
                    A.stride(0), B, B.shape[2], B.stride(0), 0.0, Y, case["n"], Y.stride(0), case["batch"],
                    prec=case["prec"])
    elif kind == "cholesky":
        return {"info": T.tdvp_cholesky(ctx, s["G"], s["L"], s["Linv"]), "L": s["L"], "Linv": s["Linv"]}
    elif kind == "eigh":
        return {"lam": T.tdvp_eigh(ctx, s["G"], s["rows"]), "rows": s["rows"]}
    else:
        T.tdvp_sweep(ctx, [s["psi"]], [s["H"]], case["dt"])
        m = T.tdvp_measure(ctx, [s["psi"]], [s["H"]])[0]
        return {"energy": m["energy"], "norm": m["norm"], "sz": m["sz"], "tensors": T.tdvp_mps_to_host(s["psi"])}
    return s["Y"]


# --------------------------------------------------------------- 64 bits
def _apply_site(W, X, transposed=False):
    """out[x, s', be, y] = sum W[al, be, s', s] X[x, al, s, y], or with al and be exchanged"""
    out = torch.zeros(X.shape[0], 2, W.shape[0] if transposed else W.shape[1], X.shape[3], dtype=X.dtype, device=X.device)
    for al, be, sp, sk in np.argwhere(W != 0):
        i, o = (be, al) if transposed else (al, be)
        out[:, sp, o] += complex(W[al, be, sp, sk]) * X[:, i, sk]
    return out


def _heff(L, W, Rt, C):
    ml, wl, _ = L.shape
    mr = Rt.shape[1]
    t1 = (L.reshape(-1, ml) @ C.reshape(ml, 2 * mr)).reshape(ml, wl, 2, mr)
    return (_apply_site(W, t1).reshape(2 * ml, -1) @ Rt.reshape(-1, mr)).reshape(ml, 2, mr)


def _keff(L, Rt, X):
    return (L.reshape(-1, L.shape[2]) @ X).reshape(L.shape[0], -1) @ Rt.reshape(-1, Rt.shape[2])


def _env_left(L, W, A):
    ml, wl, _ = L.shape
    mr = A.shape[2]
    t1 = (L.reshape(-1, ml) @ A.reshape(ml, 2 * mr)).reshape(ml, wl, 2, mr)
    return (A.reshape(2 * ml, mr).mH @ _apply_site(W, t1).reshape(2 * ml, -1)).reshape(mr, W.shape[1], mr)


def _env_right(Rt, W, B):
    ml, mr = B.shape[0], B.shape[2]
    u1 = torch.stack([B.reshape(2 * ml, mr) @ Rt[be] for be in range(W.shape[1])])       # [be, (a, s), b']
    u1 = u1.reshape(-1, ml, 2, mr).permute(1, 0, 2, 3)                                    # [a, be, s, b']
    u2 = _apply_site(W, u1, transposed=True).permute(2, 0, 1, 3).reshape(-1, 2 * mr)       # [(al, a), (s', b')]
    return (u2 @ B.reshape(ml, 2 * mr).mH).reshape(W.shape[0], ml, ml)


def _ladder_mpo(n, couplings):
    """Site tensors of sum S_i . S_j, three channels for each open coupling"""
    sp, sm, sz = np.array([[0, 1], [0, 0]]), np.array([[0, 0], [1, 0]]), np.array([[0.5, 0], [0, -0.5]])
    start, close = (sp, sm, sz), (0.5 * sm, 0.5 * sp, sz)
    opened = [[c for c in couplings if c[0] < b <= c[1]] for b in range(n + 1)]
    sites = []
    for i in range(n):
        left, right = opened[i], opened[i + 1]
        w = np.zeros((2 + 3 * len(left), 2 + 3 * len(right), 2, 2), dtype=np.complex128)
        w[0, 0] = w[-1, -1] = np.eye(2)
        for k, c in enumerate(left):
            for t in range(3):
                if c[1] == i:
                    w[1 + 3 * k + t, -1] = close[t]
                else:
                    w[1 + 3 * k + t, 1 + 3 * right.index(c) + t] = np.eye(2)
        for k, c in enumerate(right):
            if c[0] == i:
                for t in range(3):
                    w[0, 1 + 3 * k + t] = start[t]
        sites.append(w)
    sites[0], sites[-1] = sites[0][:1], sites[-1][:, -1:]
    return sites


def _exp_krylov(mv, x, z):
    """exp(z H) x by Lanczos with full reorthogonalisation, to 1e-15"""
    nrm = torch.linalg.vector_norm(x)
    V, alpha, beta = [x.reshape(-1) / nrm], [], []
    while True:
        w = mv(V[-1].reshape(x.shape)).reshape(-1)
        basis = torch.stack(V)
        alpha.append(float(torch.vdot(V[-1], w).real))
        for _ in range(2):
            w = w - basis.T @ (basis.conj() @ w)
        e, u = np.linalg.eigh(np.diag(alpha) + np.diag(beta, 1) + np.diag(beta, -1))
        c = u @ (np.exp(z * e) * u[0])
        b = float(torch.linalg.vector_norm(w))
        if b * abs(c[-1]) < 1e-15 or len(V) == 60 or b < 1e-14 * max(map(abs, alpha)):
            break
        beta.append(b)
        V.append(w / b)
    return nrm * (torch.from_numpy(c).to(basis) @ basis).reshape(x.shape)


def _exact_sweep(case, seed):
    n, z = 2 * case["legs"], -0.5j * case["dt"]
    W = _ladder_mpo(n, ladder_couplings(case["legs"]))
    M = [torch.from_numpy(t).cuda() for t in _chain_state(case, seed)]
    one = torch.ones(1, 1, 1, dtype=torch.complex128, device="cuda")
    L, R = [one] + [None] * n, [None] * n + [one]
    for i in range(n - 1, 0, -1):
        R[i] = _env_right(R[i + 1], W[i], M[i])
    for i in range(n):
        step = z if i < n - 1 else 2 * z
        M[i] = _exp_krylov(lambda c: _heff(L[i], W[i], R[i + 1], c), M[i], step)
        if i < n - 1:
            a, _, b = M[i].shape
            q, r = torch.linalg.qr(M[i].reshape(2 * a, b).cpu())
            M[i], r = q.cuda().reshape(a, 2, -1), r.cuda()
            L[i + 1] = _env_left(L[i], W[i], M[i])
            r = _exp_krylov(lambda x: _keff(L[i + 1], R[i + 1], x), r, -z)
            M[i + 1] = (r @ M[i + 1].reshape(r.shape[1], -1)).reshape(-1, 2, M[i + 1].shape[2])
    for i in range(n - 1, 0, -1):
        a, _, b = M[i].shape
        q, r = torch.linalg.qr(M[i].reshape(a, 2 * b).mH.cpu())
        M[i], r = q.mH.cuda().reshape(-1, 2, b), r.mH.cuda()
        R[i] = _env_right(R[i + 1], W[i], M[i])
        r = _exp_krylov(lambda x: _keff(L[i], R[i], x), r.contiguous(), -z)
        M[i - 1] = (M[i - 1].reshape(-1, r.shape[0]) @ r).reshape(M[i - 1].shape[0], 2, -1)
        M[i - 1] = _exp_krylov(lambda c: _heff(L[i - 1], W[i - 1], R[i], c), M[i - 1], z)
    norm2 = float(torch.vdot(M[0].reshape(-1), M[0].reshape(-1)).real)
    energy = float(torch.vdot(M[0].reshape(-1), _heff(L[0], W[0], R[1], M[0]).reshape(-1)).real) / norm2
    sz, c = [], M[0]
    for i in range(n):     # move the centre along, read S^z off it
        p = c.abs().square().sum(dim=(0, 2))
        sz.append(0.5 * float(p[0] - p[1]) / norm2)
        if i < n - 1:
            r = torch.linalg.qr(c.reshape(-1, c.shape[2]).cpu())[1].cuda()
            c = (r @ M[i + 1].reshape(r.shape[1], -1)).reshape(-1, 2, M[i + 1].shape[2])
    return {"energy": energy, "norm": math.sqrt(norm2), "sz": np.array(sz), "tensors": None}


def exact(case, seed):
    kind = case["kind"]
    if kind == "sweep":      # the tensors depend on the gauge; what is measured does not
        return _exact_sweep(case, seed)
    if kind == "cholesky":
        low = torch.linalg.cholesky(_gram(case, seed).cpu())
        eye = torch.eye(case["n"], dtype=low.dtype)
        return {"info": None, "L": low, "Linv": torch.linalg.solve_triangular(low, eye, upper=False)}
    if kind == "eigh":       # eigenvectors have a free phase
        return {"lam": np.linalg.eigvalsh(_gram(case, seed).cpu().numpy())[::-1].copy(), "rows": None}
    if kind == "gemm":
        A, B = (x.to(torch.complex128) for x in _gemm_operands(case, seed))
        op = {"N": lambda x: x, "T": lambda x: x.mT, "C": lambda x: x.mH, "R": lambda x: x.conj()}
        return torch.stack([op[case["opa"]](A[b]).resolve_conj().contiguous() @ op[case["opb"]](B[b]).resolve_conj().contiguous()
                            for b in range(case["batch"])])
    o = {k: v.to(torch.complex128) if isinstance(v, torch.Tensor) else v for k, v in _operands(case, seed).items()}
    if kind == "keff":
        return _keff(o["L"], o["Rt"], o["C"])
    if kind == "env_left":
        return _env_left(o["L"], o["W"], o["C"])
    if kind == "env_right":
        return _env_right(o["Rt"], o["W"], o["C"])
    return _heff(o["L"], o["W"], o["Rt"], o["C"])


# ------------------------------------------------------------ minimal work
def work(case):
    """Each operand read once and each result written once; 8 operations for a
    complex multiply-add of the terms that are not zero by structure."""
    kind = case["kind"]
    if kind == "gemm":
        m, n, k, b = (case[x] for x in ("m", "n", "k", "batch"))
        cb = 16 if case["prec"] == "fp64" else 8
        return dict(bytes=cb * b * (m * k + k * n + m * n), flops=8 * b * m * n * k)
    if kind == "cholesky":      # factor and inverse, n^3 / 6 multiply-adds each
        n = case["n"]
        return dict(bytes=16 * 3 * n * n, flops=8 * n ** 3 / 3)
    if kind == "eigh":          # reduction 4/3, its back transformation 4/3, vectors of the tridiagonal matrix (real) 4/3
        n = case["n"]
        return dict(bytes=16 * 2 * n * n, flops=(4 + 4 + 1) * 4 * n ** 3 / 3)
    if kind == "sweep":         # both half sweeps: at least four matvecs a site and a bond, one environment update
        n, flops, size = 2 * case["legs"], 0.0, 0
        d = [min(case["chi"], 2 ** min(i, n - i)) for i in range(n + 1)]
        for i in range(n):
            w = [8 if 0 < b < n else 1 for b in (i, i + 1)]
            flops += 2 * 5 * 8 * 2 * d[i] * d[i + 1] * (d[i] * w[0] + d[i + 1] * w[1]) + 2 * 4 * 8 * d[i + 1] ** 3 * w[1] * 2
            size += d[i] * 2 * d[i + 1]
        return dict(bytes=16 * 3 * size, flops=flops)
    ml, mr, wl, wr = (case[x] for x in ("ml", "mr", "wl", "wr"))
    cb = 16 if case["prec"] == "fp64" else 8
    nnz = int(np.count_nonzero(mpo_site(wl, wr, 0)[0]))
    left, right = ml * wl * ml, mr * wr * mr
    if kind == "keff":
        return dict(bytes=cb * (left + right + 2 * ml * mr), flops=8 * ml * mr * (ml * wl + mr * wr))
    if kind in ("env_left", "env_right"):
        return dict(bytes=cb * (left + right + 2 * ml * mr), flops=8 * (2 * ml * mr * (ml * wl + mr * wr) + nnz * ml * mr))
    if kind == "heff":
        return dict(bytes=cb * (left + right + 4 * ml * mr), flops=8 * (2 * ml * mr * (ml * wl + mr * wr) + nnz * ml * mr))
    # with charges: the blocks alone
    ql, qr = charges(ml, EVEN_SECTORS), charges(mr, ODD_SECTORS)
    W, qwl, qwr = mpo_site(wl, wr, 0)
    nl, nr = (dict(zip(*(v.tolist() for v in np.unique(q, return_counts=True)))) for q in (ql, qr))
    macs = entries = 0
    for qa in qwl.tolist():      # T1[a', al, s, b] = L[a', al, a] C[a, s, b]
        for a2, n2 in nl.items():
            n1 = nl.get(a2 - qa, 0)
            entries += n2 * n1
            macs += n2 * n1 * sum(nr.get(a2 - qa + s, 0) for s in (1, -1))
    for qb in qwr.tolist():      # Y[a', s', b'] = T2[a', s', be, b] Rt[be, b, b']
        for b2, n2 in nr.items():
            n1 = nr.get(b2 - qb, 0)
            entries += n2 * n1
            macs += n2 * n1 * sum(nl.get(b2 - s, 0) for s in (1, -1))
    site = sum(n * nr.get(q + s, 0) for q, n in nl.items() for s in (1, -1))
    return dict(bytes=cb * (entries + 2 * site), flops=8 * macs)
