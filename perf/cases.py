"""Performance cases of the library: what a program built on it calls, at the
sizes such programs have.

Every case is a dict of plain values; ``kind`` names the entry point:

* ``gemm``      - Context.dgemm, emulated (slices 2..8) or native FP64
  (slices 0), with transposes, alpha / beta and ragged sizes;
* ``dense``     - HeffPlan.apply of a dense two-site H_eff;
* ``sparse``    - HeffPlan.apply of a block-sparse H_eff (symmetry sectors);
* ``davidson``  - a whole Davidson solve (solver made, run, Ritz vector read),
  what one site update of a DMRG sweep does with its plan;
* ``lanczos``   - the same with Lanczos;
* ``truncate``  - rho = psi psi^T, its dominant eigenvectors U and the
  truncated tensor U U^T psi;
* ``renormalize`` - U^T O_k U of a list of block operators.

Element distributions follow workloads.py: N(0,1) 2^u with u uniform in
[-U, U] for operators and tensors, GOE-like operators with a planted
reference state for the eigensolvers, a planted Schmidt spectrum for the
truncation.
"""
import math

import numpy as np
import torch

from paper_2510_04795_amd import ozaki

DEV = "cuda:0"

# Largest product a draw may give (its FP64 operations): no drawn case costs
# more than the listed ones.
_MAX_GEMM = 2.0 * 4096 ** 3


def listed():
    return [
        # One block product of a small sector: launches and latency count.
        {"name": "gemm_tiny", "kind": "gemm", "m": 96, "n": 160, "k": 200, "transa": "N", "transb": "N",
         "slices": 6, "ndiag": 6, "alpha": 1.0, "beta": 0.0},
        # The plain 512^3 product at the width that keeps FP64 accuracy.
        {"name": "gemm_512", "kind": "gemm", "m": 512, "n": 512, "k": 512, "transa": "N", "transb": "N",
         "slices": 7, "ndiag": 8, "alpha": 1.0, "beta": 0.0},
        # A ragged accumulating product with a transposed operand, as a
        # program contracting tensors of odd bond dimensions issues it.
        {"name": "gemm_ragged", "kind": "gemm", "m": 1021, "n": 1531, "k": 2777, "transa": "T", "transb": "N",
         "slices": 7, "ndiag": 7, "alpha": 0.5, "beta": 1.0},
        # The headline product at equal error.
        {"name": "gemm_8192", "kind": "gemm", "m": 8192, "n": 8192, "k": 8192, "transa": "N", "transb": "N",
         "slices": 7, "ndiag": 7, "alpha": 1.0, "beta": 0.0},
        # Native FP64 where performant dispatch takes it: the small product.
        {"name": "fp64_512", "kind": "gemm", "m": 512, "n": 512, "k": 512, "transa": "N", "transb": "N",
         "slices": 0, "ndiag": 0, "alpha": 1.0, "beta": 0.0},
        # Native FP64 at an ordinary size, second operand transposed (rho, R^T).
        {"name": "fp64_2048", "kind": "gemm", "m": 2048, "n": 2048, "k": 2048, "transa": "N", "transb": "T",
         "slices": 0, "ndiag": 0, "alpha": 1.0, "beta": 0.0},
        # Dense two-site H_eff: the matvec of a large bond dimension.
        {"name": "dense_1024", "kind": "dense", "d": 1024, "phys": 16, "kop": 32, "slices": 6},
        # Block-sparse H_eff: 40 sectors, 2000 operator triples.
        {"name": "sparse_40", "kind": "sparse", "sectors": 40, "triples": 2000, "median": 200.0, "kop": 64,
         "layout": 0, "slices": 6},
        # One Davidson solve of a site update.
        {"name": "davidson_1024", "kind": "davidson", "d": 1024, "kop": 32, "slices": 6, "m_max": 32, "tol": 1e-8},
        # One Lanczos solve on a small site: latency of a whole small call.
        {"name": "lanczos_96", "kind": "lanczos", "d": 96, "kop": 8, "slices": 6, "m_max": 32, "tol": 1e-5},
        # Truncation of a two-site tensor to a quarter of its states, FP64.
        {"name": "truncate_2048", "kind": "truncate", "n": 2048, "keep": 512, "slices": 0},
        # Renormalisation of the block operators into the kept basis.
        {"name": "renormalize_2048", "kind": "renormalize", "n": 2048, "keep": 512, "count": 16, "slices": 7},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["gemm", "gemm", "fp64", "dense", "sparse", "davidson", "lanczos", "truncate", "renormalize"])
    if kind in ("gemm", "fp64"):
        while True:
            m, n, k = (_log(rng, 32, 8192) for _ in range(3))
            if 2.0 * m * n * k <= _MAX_GEMM:
                break
        s = 0 if kind == "fp64" else rng.choice([4, 5, 6, 6, 7, 7, 8])
        acc = rng.random() < 0.3
        return {"kind": "gemm", "m": m, "n": n, "k": k, "transa": rng.choice("NT"), "transb": rng.choice("NT"),
                "slices": s, "ndiag": s + (1 if s and rng.random() < 0.3 else 0),
                "alpha": 0.5 if acc else 1.0, "beta": 1.0 if acc else 0.0}
    if kind == "dense":
        return {"kind": "dense", "d": _log(rng, 48, 768), "phys": rng.choice([1, 4, 16]), "kop": rng.randint(2, 32),
                "slices": rng.choice([0, 5, 6, 6, 7, 8])}
    if kind == "sparse":
        return {"kind": "sparse", "sectors": rng.randint(8, 40), "triples": _log(rng, 60, 1500),
                "median": float(_log(rng, 40, 200)), "kop": rng.randint(8, 64), "layout": rng.randint(1, 1000000),
                "slices": rng.choice([0, 5, 6, 6, 7, 8])}
    if kind in ("davidson", "lanczos"):
        return {"kind": kind, "d": _log(rng, 32, 768), "kop": rng.randint(4, 24),
                "slices": rng.choice([0, 5, 6, 6, 7]), "m_max": rng.choice([16, 32]),
                "tol": rng.choice([1e-5, 1e-8])}
    n = _log(rng, 96, 1600)
    if kind == "truncate":
        return {"kind": kind, "n": n, "keep": max(8, n // rng.randint(4, 6)), "slices": rng.choice([0, 0, 7, 8])}
    return {"kind": kind, "n": n, "keep": max(8, n // rng.randint(2, 6)), "count": rng.randint(2, 16),
            "slices": rng.choice([0, 0, 6, 7, 8])}


# ---- inputs -------------------------------------------------------------------
def _rng(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + 17)
    return g


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float64)


def _wide(g, u, *shape):
    e = torch.randint(-u, u + 1, shape, generator=g, device=DEV, dtype=torch.int32)
    return torch.ldexp(_normal(g, *shape), e)


def _sym(x):
    return (x + x.transpose(-1, -2)) * 0.5


def _gemm_inputs(case, seed):
    g = _rng(seed)
    m, n, k = case["m"], case["n"], case["k"]
    A = _wide(g, 10, *((k, m) if case["transa"] == "T" else (m, k)))
    B = _wide(g, 10, *((n, k) if case["transb"] == "T" else (k, n)))
    return A, B, (_wide(g, 10, m, n) if case["beta"] else None)


def _dense_inputs(case, seed):
    g = _rng(seed)
    d, p, kop = case["d"], case["phys"], case["kop"]
    L = torch.stack([_sym(_wide(g, 8, d, d)) for _ in range(kop)])
    R = torch.stack([_sym(_wide(g, 8, d, d)) for _ in range(kop)])
    return L, R, _wide(g, 8, d, p, d)


def _dense_layout(d, phys, kop):
    key = [x for k in range(kop) for x in (k, 0, 0)]
    off = [k * d * d for k in range(kop)]
    layout = {"left_dim": [d], "right_dim": [d], "phys": phys, "psi_lr": [0, 0], "psi_offset": [0],
              "L_key": key, "L_offset": off, "R_key": key, "R_offset": off}
    return layout, [(k, 0, 0, 0, 0, 1.0) for k in range(kop)]


def _sparse_structure(case):
    """Sector sizes, the blocks of psi and the triples, from the case alone
    (log-normal sizes, mask density 0.12, sector moves of at most two)."""
    rng = np.random.default_rng(case["layout"])
    q, kop = case["sectors"], case["kop"]
    dims = np.clip(np.rint(np.exp(math.log(case["median"]) + 0.8 * rng.standard_normal(q))), 16, 1500).astype(int)
    mask = rng.random((q, q)) < 0.12
    mask[np.arange(q), rng.permutation(q)] = True
    blocks = sorted((int(a), int(b)) for a, b in np.argwhere(mask))
    near = {b: [c for c in blocks if abs(c[0] - b[0]) <= 2 and abs(c[1] - b[1]) <= 2] for b in blocks}
    room = kop * sum(len(v) for v in near.values())
    seen = {}
    while len(seen) < min(case["triples"], room // 2):
        op = int(rng.integers(0, kop))
        li, ri = blocks[int(rng.integers(0, len(blocks)))]
        lo, ro = near[(li, ri)][int(rng.integers(0, len(near[(li, ri)])))]
        seen[(op, lo, li, ri, ro)] = None
    triples = [t + (1.0,) for t in seen]
    return [int(x) for x in dims], blocks, triples


def _offsets(sizes):
    off, at = [], 0
    for s in sizes:
        off.append(at)
        at += s
    return off, at


def _sparse_inputs(case, seed):
    dims, blocks, triples = _sparse_structure(case)
    lk = sorted({t[:3] for t in triples})
    rk = sorted({(t[0], t[4], t[3]) for t in triples})
    poff, pn = _offsets([dims[a] * dims[b] for a, b in blocks])
    loff, ln = _offsets([dims[a] * dims[b] for _, a, b in lk])
    roff, rn = _offsets([dims[a] * dims[b] for _, a, b in rk])
    layout = {"left_dim": dims, "right_dim": dims, "phys": 1, "psi_lr": [x for b in blocks for x in b],
              "psi_offset": poff, "L_key": [x for k in lk for x in k], "L_offset": loff,
              "R_key": [x for k in rk for x in k], "R_offset": roff}
    g = _rng(seed)
    return layout, triples, _wide(g, 12, ln), _wide(g, 12, rn), _wide(g, 12, pn)


def _solver_inputs(case, seed):
    """GOE-like operator pairs scaled to a total spectral norm of about 10,
    a reference state of energy -30 and a start vector near it."""
    g = _rng(seed)
    d, kop = case["d"], case["kop"]
    c = 1.0 / (2.0 * math.sqrt(d))
    L, R = (_sym(_normal(g, kop, d, d)) * c for _ in range(2))
    v = _normal(g, d, d)
    for _ in range(20):
        v = v / torch.linalg.vector_norm(v)
        w = torch.zeros_like(v)
        for k in range(kop):
            w += L[k] @ v @ R[k]
        nu, v = torch.linalg.vector_norm(w), w
    s = torch.sqrt(10.0 / nu)
    L, R = (L * s).contiguous(), (R * s).contiguous()
    delta = torch.zeros(d, d, dtype=torch.float64, device=DEV)
    delta[0, 0] = -30.0
    hdiag = torch.zeros_like(delta)
    for k in range(kop):
        hdiag += torch.outer(torch.diagonal(L[k]), torch.diagonal(R[k]))
    hdiag += delta
    r = _normal(g, d * d)
    x0 = 0.1 * r / torch.linalg.vector_norm(r)
    x0[0] += 1.0
    return L, R, delta.reshape(-1), hdiag.reshape(-1), x0 / torch.linalg.vector_norm(x0)


def _orthonormal(g, rows, cols):
    q, r = torch.linalg.qr(_normal(g, rows, cols))
    return (q * torch.sign(torch.diagonal(r))).contiguous()


def _schmidt(case, seed):
    """Orthonormal left and right vectors and the squared Schmidt values."""
    g = _rng(seed)
    n = case["n"]
    w = torch.exp(-torch.arange(n, device=DEV, dtype=torch.float64) / (n / 64.0))
    return _orthonormal(g, n, n), _orthonormal(g, n, n), w / w.sum()


def _renorm_inputs(case, seed):
    g = _rng(seed)
    n = case["n"]
    U = _orthonormal(g, n, case["keep"])
    return U, [_sym(_normal(g, n, n)) / math.sqrt(n) for _ in range(case["count"])]


# ---- the cases ------------------------------------------------------------------
def prepare(case, seed):
    kind, s = case["kind"], case["slices"]
    ctx = ozaki.Context(0)
    st = {"case": case, "ctx": ctx}
    if kind == "gemm":
        A, B, C = _gemm_inputs(case, seed)
        st.update(A=A, B=B, C0=C, C=torch.empty(case["m"], case["n"], dtype=torch.float64, device=DEV),
                  ws=ctx.workspace(case["m"], case["n"], case["k"], s, case["ndiag"]))
    elif kind == "dense":
        L, R, psi = _dense_inputs(case, seed)
        layout, triples = _dense_layout(case["d"], case["phys"], case["kop"])
        st.update(psi=psi.reshape(-1), sigma=torch.empty(psi.numel(), dtype=torch.float64, device=DEV),
                  plan=ozaki.HeffPlan(ctx, layout, L.reshape(-1), R.reshape(-1), triples, slices=s))
    elif kind == "sparse":
        layout, triples, L, R, psi = _sparse_inputs(case, seed)
        st.update(psi=psi, sigma=torch.empty_like(psi), plan=ozaki.HeffPlan(ctx, layout, L, R, triples, slices=s))
    elif kind in ("davidson", "lanczos"):
        L, R, delta, hdiag, x0 = _solver_inputs(case, seed)
        layout, triples = _dense_layout(case["d"], 1, case["kop"])
        st.update(hdiag=hdiag, x0=x0,
                  plan=ozaki.HeffPlan(ctx, layout, L.reshape(-1), R.reshape(-1), triples, diag=delta, slices=s))
    elif kind == "truncate":
        X, Y, w = _schmidt(case, seed)
        st.update(psi=((X * torch.sqrt(w)) @ Y.T).contiguous(), eig=ozaki.RdmEig(ctx, case["n"], s))
    else:
        U, ops = _renorm_inputs(case, seed)
        st.update(U=U, ops=ops)
    return st


def run(st):
    case, ctx = st["case"], st["ctx"]
    kind, s = case["kind"], case["slices"]
    if kind == "gemm":
        C = st["C"]
        if case["beta"]:
            C.copy_(st["C0"])  # the tensor the product is added to
        return ctx.dgemm(st["A"], st["B"], slices=s, ndiag=case["ndiag"], alpha=case["alpha"], beta=case["beta"],
                         C=C, transa=case["transa"], transb=case["transb"], workspace=st["ws"])
    if kind in ("dense", "sparse"):
        return st["plan"].apply(st["psi"], st["sigma"])
    if kind in ("davidson", "lanczos"):
        if kind == "davidson":
            solver = ozaki.Davidson(ctx, st["plan"], st["hdiag"], st["x0"], m_max=case["m_max"], tol=case["tol"])
        else:
            solver = ozaki.Lanczos(ctx, st["plan"], st["x0"], m_max=case["m_max"], tol=case["tol"])
        theta = solver.run()[0]
        x = solver.vector()
        solver.close()
        return {"theta": theta, "x": x}
    if kind == "truncate":
        # eigenvectors have no sign of their own: the truncated tensor does
        # not depend on it
        psi = st["psi"]
        rho = ctx.dgemm(psi, psi, slices=s, transb="T")
        evals, U, info = st["eig"].solve(rho, case["keep"])
        site = ctx.dgemm(U, psi, slices=s, transa="T")
        return {"evals": evals, "trace": info.trace, "psi": ctx.dgemm(U, site, slices=s)}
    return ctx.renormalize(st["U"], st["ops"], slices=s)


def _pairs(s, g):
    """Slice pairs (s, t) with s + t < g; one FP64 product when native."""
    return sum(1 for a in range(s) for b in range(s) if a + b < (g or s)) if s else 1


def work(case):
    """Bytes: inputs read once, outputs written once, in FP64.  flops: 2mnk
    per native product, 2mnk integer operations per kept slice pair when
    emulated."""
    kind, p = case["kind"], _pairs(case["slices"], case.get("ndiag", 0))
    if kind == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": 8.0 * (m * k + k * n + m * n * (3 if case["beta"] else 1)), "flops": 2.0 * m * n * k * p}
    if kind == "dense":
        d, f, kop = case["d"], case["phys"], case["kop"]
        return {"bytes": 8.0 * (2 * kop * d * d + 2 * d * d * f), "flops": 4.0 * d ** 3 * f * kop * p}
    if kind == "sparse":
        dims, blocks, triples = _sparse_structure(case)
        lk = {t[:3] for t in triples}
        rk = {(t[0], t[4], t[3]) for t in triples}
        first = {t[:4] for t in triples}
        el = sum(dims[a] * dims[b] for _, a, b in lk) + sum(dims[a] * dims[b] for _, a, b in rk)
        el += 2 * sum(dims[a] * dims[b] for a, b in blocks)
        fl = sum(2.0 * dims[lo] * dims[li] * dims[ri] for _, lo, li, ri in first)
        fl += sum(2.0 * dims[lo] * dims[ri] * dims[ro] for _, lo, _, ri, ro, _ in triples)
        return {"bytes": 8.0 * el, "flops": fl * p}
    if kind in ("davidson", "lanczos"):
        # matvecs of a typical solve (12) and the basis vectors they add
        d, kop = case["d"], case["kop"]
        return {"bytes": 12 * 8.0 * (2 * kop * d * d + 16 * d * d), "flops": 12 * 4.0 * d ** 3 * kop * p}
    n, keep = case["n"], case["keep"]
    if kind == "truncate":
        return {"bytes": 8.0 * (2 * n * n + keep), "flops": (2.0 * n ** 3 + 4.0 * n * n * keep) * p + 4.0 / 3 * n ** 3}
    return {"bytes": 8.0 * (n * keep + case["count"] * (n * n + keep * keep)),
            "flops": case["count"] * 2.0 * (n * n * keep + n * keep * keep) * p}


def exact(case, seed):
    kind = case["kind"]
    if kind == "gemm":
        A, B, C = _gemm_inputs(case, seed)
        P = (A.T if case["transa"] == "T" else A) @ (B.T if case["transb"] == "T" else B)
        return case["alpha"] * P + (case["beta"] * C if case["beta"] else 0.0)
    if kind == "dense":
        L, R, psi = _dense_inputs(case, seed)
        d, f = case["d"], case["phys"]
        out = torch.zeros(d * f, d, dtype=torch.float64, device=DEV)
        for k in range(case["kop"]):
            out += (L[k] @ psi.reshape(d, f * d)).reshape(d * f, d) @ R[k].T
        return out.reshape(-1)
    if kind == "sparse":
        layout, triples, L, R, psi = _sparse_inputs(case, seed)
        dims, blocks, _ = _sparse_structure(case)

        def view(x, key, off):
            n = len(key) // len(off)
            return {tuple(key[n * i:n * i + n]): x[o:o + dims[key[n * i + n - 2]] * dims[key[n * i + n - 1]]]
                    .view(dims[key[n * i + n - 2]], dims[key[n * i + n - 1]]) for i, o in enumerate(off)}

        lv, rv = view(L, layout["L_key"], layout["L_offset"]), view(R, layout["R_key"], layout["R_offset"])
        out = torch.zeros_like(psi)
        pv, ov = (view(x, layout["psi_lr"], layout["psi_offset"]) for x in (psi, out))
        for op, lo, li, ri, ro, _ in triples:
            ov[(lo, ro)] += (lv[(op, lo, li)] @ pv[(li, ri)]) @ rv[(op, ro, ri)].T
        return out
    if kind in ("davidson", "lanczos"):
        # the lowest eigenvalue by Lanczos with full reorthogonalisation; the
        # vector is only as exact as the residual the solver stops at
        L, R, delta, _, x = _solver_inputs(case, seed)
        d = case["d"]
        Q, T = [x], np.zeros((60, 60))
        for j in range(60):
            w = delta * Q[j]
            v = Q[j].view(d, d)
            for k in range(case["kop"]):
                w = w + (L[k] @ v @ R[k].T).reshape(-1)
            T[j, j] = float(torch.dot(w, Q[j]))
            B = torch.stack(Q)
            for _ in range(2):
                w = w - B.T @ (B @ w)
            b = float(torch.linalg.vector_norm(w))
            e, y = np.linalg.eigh(T[:j + 1, :j + 1])
            if b * abs(y[-1, 0]) < 1e-11 or j == 59:
                break
            T[j, j + 1] = T[j + 1, j] = b
            Q.append(w / b)
        return {"theta": float(e[0]), "x": None}
    if kind == "truncate":
        # the planted decomposition: closed forms of all three
        X, Y, w = _schmidt(case, seed)
        d = case["keep"]
        return {"evals": w[:d].contiguous(), "trace": float(w.sum()),
                "psi": (X[:, :d] * torch.sqrt(w[:d])) @ Y[:, :d].T}
    U, ops = _renorm_inputs(case, seed)
    return [U.T @ (o @ U) for o in ops]
