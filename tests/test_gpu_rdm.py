"""GPU truncation and renormalisation: the block-Jacobi RDM eigensolver
against LAPACK's eigh (eigenvalues, residuals, orthogonality, kept subspace)
in native and emulated arithmetic, the truncation of a planted two-site
tensor, and ozaki_renormalize bit-exact against the oracle's GEMM
composition (emulated) or within the FP64 GEMM bound (native)."""
import numpy as np
import pytest

import oracle
from paper_2510_04795_amd import workloads as wl
from tests.helpers import assert_bitexact

pytestmark = pytest.mark.gpu
U64 = 2.0 ** -53


@pytest.fixture(scope="module")
def oz():
    import torch
    from paper_2510_04795_amd import ozaki
    torch.cuda.init()
    ctx = ozaki.Context(0)
    yield ozaki, ctx, torch
    ctx.close()


def dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def u_eff(S):
    return U64 if S == 0 else max(U64, 2.0 ** (1 - 8 * S))


def solve(oz, A, S=0, nev=None, **kw):
    ozaki, ctx, torch = oz
    eig = ozaki.RdmEig(ctx, A.shape[0], S)
    try:
        w, Z, info = eig.solve(dev(torch, A), nev, **kw)
        return w.cpu().numpy(), Z.cpu().numpy(), info
    finally:
        eig.close()


def check_eigenpairs(A, w, Z, S, slack=1.0):
    """Eigenvalues against LAPACK, residual and orthogonality, all within
    64 sqrt(n) u |A|_2 (u of the arithmetic in use)."""
    n = A.shape[0]
    nev = w.size
    ref = oracle.rdm_eigh(A, nev)[0]
    norm = max(np.linalg.norm(A, 2), np.finfo(float).tiny)
    tol = slack * 64 * np.sqrt(n) * u_eff(S)
    assert np.all(np.diff(w) <= 0), "eigenvalues not in decreasing order"
    assert np.max(np.abs(w - ref)) <= tol * norm, np.max(np.abs(w - ref)) / norm
    res = np.linalg.norm(A @ Z - Z * w, axis=0)
    assert np.max(res) <= tol * norm, np.max(res) / norm
    assert np.max(np.abs(Z.T @ Z - np.eye(nev))) <= tol, np.max(np.abs(Z.T @ Z - np.eye(nev)))


def wishart(n, r=None, seed=0):
    B = np.random.default_rng(seed).standard_normal((n, n if r is None else r))
    return B @ B.T / n


@pytest.mark.parametrize("n", [1, 40, 200, 513])
def test_fp64_wishart(oz, n):
    A = wishart(n, seed=n)
    w, Z, info = solve(oz, A)
    assert info.status == 1 and info.sweeps >= 1
    check_eigenpairs(A, w, Z, 0)
    assert abs(info.trace - np.trace(A)) <= 1e-12 * abs(np.trace(A))


@pytest.mark.parametrize("n", [64, 300])
def test_fp64_planted_rdm(oz, n):
    """An RDM whose spectrum decays to e^-64: the clustered tail of tiny
    eigenvalues converges slowly (linear phase of cyclic Jacobi), but the
    kept quarter must be resolved to FP64 accuracy within the sweep limit."""
    t = wl.two_site_psi(n, tau=n / 64.0, seed=1)
    A = t.psi @ t.psi.T
    w, Z, info = solve(oz, A, nev=n // 4)
    assert info.status in (1, 3)
    check_eigenpairs(A, w, Z, 0)
    assert np.max(np.abs(w - t.schmidt[: n // 4] ** 2)) <= 64 * np.sqrt(n) * U64 * w[0]


@pytest.mark.parametrize("S", [7, 5, 4, 3])
def test_emulated_accuracy_follows_slices(oz, S):
    """With the Gram and rotation GEMMs emulated, the eigenpairs keep the
    accuracy of the emulation's 8S - 1 bits."""
    A = wishart(256, seed=2)
    w, Z, info = solve(oz, A, S)
    assert info.status in (1, 2)
    check_eigenpairs(A, w, Z, S)


@pytest.mark.parametrize("seed", range(8))
def test_random_symmetric(oz, seed):
    """Seeded random symmetric matrices: sizes 2..300 (off the 32-row
    blocks), positive semidefinite of full or deficient rank, or indefinite;
    a random number of wanted eigenpairs; FP64 or S = 4..7.  Eigenvalues,
    residuals and orthogonality within the bound of the arithmetic."""
    rng = np.random.default_rng(700 + seed)
    n = int(rng.integers(2, 301))
    kind = int(rng.integers(0, 3))
    if kind == 0:
        A = wishart(n, seed=800 + seed)
    elif kind == 1:
        A = wishart(n, r=int(rng.integers(1, n + 1)), seed=800 + seed)
    else:
        X = np.random.default_rng(800 + seed).standard_normal((n, n))
        A = (X + X.T) / 2
    nev = int(rng.integers(1, n + 1))
    S = int(rng.choice([0, 4, 5, 6, 7]))
    w, Z, info = solve(oz, A, S, nev=nev)
    assert info.status in (1, 2, 3), (seed, n, kind, nev, S, info.status)
    check_eigenpairs(A, w, Z, S)


@pytest.mark.parametrize("n", [65, 128, 129, 320])
@pytest.mark.parametrize("kind", ["graded", "singular_shift", "rank_one"])
def test_qr_iteration_start(oz, n, kind):
    """Starts of the sweeps from QR iteration around the 64-column panels: a
    graded density matrix (both steps taken); an indefinite matrix whose
    shifted copy is singular (an eigenvalue of -3e-7 |A|_F: the first
    factorisation breaks down and the sweeps start from A itself, or from a
    pass of poor orthogonality that has to be refused); rank one (all but one
    column of the shifted copy is the shift alone)."""
    rng = np.random.default_rng(n)
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    if kind == "graded":
        lam = np.exp(-np.arange(n) / (n / 64.0))
    elif kind == "rank_one":
        lam = np.zeros(n)
        lam[0] = 1.0
    else:
        lam = rng.standard_normal(n)
        lam[n // 2] = 0.0
        lam[n // 2] = -3e-7 * np.linalg.norm(lam)
    A = (Q * lam) @ Q.T
    A = 0.5 * (A + A.T)
    nev = n // 4 if kind == "graded" else n
    w, Z, info = solve(oz, A, nev=nev)
    assert info.status in (1, 2, 3)
    check_eigenpairs(A, w, Z, 0)


@pytest.mark.parametrize("n", [65, 130, 200, 330])
@pytest.mark.parametrize("nev", ["all", "few", "none"])
def test_pairs_that_rotate_nothing(oz, n, nev):
    """Nearly diagonal matrices whose couplings sit in some 32-row blocks only:
    most pairs rotate nothing in a round (their tiles and basis rows are only
    moved), next to pairs that do, on both sides of either product; every
    coupling small enough that the sweeps start from the matrix itself."""
    rng = np.random.default_rng(n)
    lam = np.sort(rng.uniform(0.5, 2.0, n))[::-1].copy()
    A = np.diag(lam)
    nb = -(-n // 32)
    for b, c in ((0, 0), (0, nb - 1), (nb // 2, nb - 1), (nb - 1, nb - 1)):
        r, q = slice(32 * b, min(32 * b + 32, n)), slice(32 * c, min(32 * c + 32, n))
        E = 1e-5 * rng.standard_normal(A[r, q].shape)
        A[r, q] += E
        A[q, r] += E.T
    A = 0.5 * (A + A.T)
    w, Z, info = solve(oz, A, nev={"all": n, "few": n // 4, "none": 1}[nev])
    assert info.status == 1
    check_eigenpairs(A, w, Z, 0)


def test_edge_matrices(oz):
    # zero matrix: all eigenvalues 0, orthonormal eigenvectors
    w, Z, info = solve(oz, np.zeros((50, 50)))
    assert np.all(w == 0) and np.max(np.abs(Z.T @ Z - np.eye(50))) < 1e-14
    # identity (one eigenvalue of multiplicity n)
    w, Z, _ = solve(oz, np.eye(70))
    assert np.max(np.abs(w - 1)) < 1e-14 and np.max(np.abs(Z.T @ Z - np.eye(70))) < 1e-14
    # diagonal with distinct entries: unit eigenvectors, sorted values
    d = np.random.default_rng(3).permutation(np.arange(1.0, 91.0))
    w, Z, info = solve(oz, np.diag(d))
    assert np.array_equal(w, np.sort(d)[::-1])
    assert np.array_equal(np.abs(Z), np.eye(90)[:, np.argsort(-d)])
    # rank-deficient: the nonzero part is resolved, the rest is ~0
    A = wishart(120, r=30, seed=4)
    w, Z, info = solve(oz, A)
    check_eigenpairs(A, w, Z, 0)
    assert np.max(np.abs(w[30:])) < 1e-13 * w[0]
    # nev = 0 and nev < n
    w, Z, _ = solve(oz, A, nev=0)
    assert w.size == 0 and Z.shape == (120, 0)
    w5, Z5, _ = solve(oz, A, nev=5)
    check_eigenpairs(A, w5, Z5, 0)


def test_errors(oz):
    ozaki, ctx, torch = oz
    for n in (0, 8193):
        with pytest.raises(ozaki.OzakiError):
            ozaki.RdmEig(ctx, n)
    with pytest.raises(ozaki.OzakiError):
        ozaki.RdmEig(ctx, 64, slices=1)
    eig = ozaki.RdmEig(ctx, 16)
    A = np.eye(16)
    A[3, 5] = np.nan
    with pytest.raises(ozaki.OzakiError):
        eig.solve(dev(torch, A))
    with pytest.raises(ozaki.OzakiError):
        eig.solve(dev(torch, np.eye(16)), 17)
    with pytest.raises(ozaki.OzakiError):
        eig.solve(dev(torch, np.eye(16)), max_sweeps=0)
    # the plan is still usable after rejected calls
    w, Z, info = eig.solve(dev(torch, np.diag(np.arange(16.0))))
    assert np.array_equal(w.cpu().numpy(), np.arange(15.0, -1.0, -1.0))
    eig.close()


def test_two_calls_share_a_plan(oz):
    ozaki, ctx, torch = oz
    eig = ozaki.RdmEig(ctx, 100, 6)
    for seed in (5, 6):
        A = wishart(100, seed=seed)
        w, Z, info = eig.solve(dev(torch, A))
        check_eigenpairs(A, w.cpu().numpy(), Z.cpu().numpy(), 6)
    eig.close()


@pytest.mark.parametrize("S", [0, 5])
def test_truncate_matches_oracle(oz, S):
    """rho is bit-exact with the oracle's (emulated) or within the FP64 GEMM
    bound; the kept subspace, eigenvalues and discarded weight agree."""
    ozaki, ctx, torch = oz
    t = wl.two_site_psi(160, 144, tau=8.0, seed=7)
    D = 40
    psi = dev(torch, t.psi)
    rho = ctx.dgemm(psi, psi, slices=S, transb="T").cpu().numpy()
    if S:
        assert_bitexact(rho, oracle.ozaki_dgemm(t.psi, t.psi, S, transb="T"), "rho")
    else:
        ap = np.abs(t.psi)
        gam = 144 * U64 / (1 - 144 * U64)
        assert np.all(np.abs(rho - t.psi @ t.psi.T) <= 2 * gam * (ap @ ap.T))
    U, w, dw, info = ozaki.truncate(ctx, psi, D, slices=S)
    U_ref, w_ref, dw_ref = oracle.truncate(t.psi, D, S=S)
    tol = 64 * np.sqrt(160) * u_eff(S)
    assert np.max(np.abs(w.cpu().numpy() - w_ref)) <= tol * w_ref[0]
    assert abs(dw - dw_ref) <= tol
    sv = np.linalg.svd(U_ref.T @ U.cpu().numpy(), compute_uv=False)
    assert np.all(np.abs(sv - 1) < 1e-8)


@pytest.mark.parametrize("S", [3, 6])
def test_renormalize_bitexact(oz, S):
    ozaki, ctx, torch = oz
    n, D = 200, 64
    ops = wl.block_operators(n, 3, seed=8)
    t = wl.two_site_psi(n, tau=10.0, seed=9)
    U = oracle.truncate(t.psi, D)[0]
    out = ctx.renormalize(dev(torch, U), [dev(torch, o) for o in ops], slices=S)
    for got, want in zip(out, oracle.renormalize(U, ops, S=S)):
        assert_bitexact(got.cpu().numpy(), want, "renormalize S=%d" % S)


@pytest.mark.parametrize("seed", range(6))
def test_renormalize_random_bitexact(oz, seed):
    """Seeded random renormalisations: n = 1..260, D = 1..n, 1 to 4
    operators with entries spread over 2^-6..2^6, a general (not orthonormal)
    U, S = 2..8 with every built ndiag: the oracle's bits."""
    ozaki, ctx, torch = oz
    rng = np.random.default_rng(900 + seed)
    n = int(rng.integers(1, 261))
    D = int(rng.integers(1, n + 1))
    k = int(rng.integers(1, 5))
    S = int(rng.integers(2, 9))
    G = int(rng.choice(sorted({S, S + 1, 2 * S - 1})))

    def spread(shape):
        return np.ldexp(rng.standard_normal(shape), rng.integers(-6, 7, size=shape))

    U = spread((n, D))
    ops = [spread((n, n)) for _ in range(k)]
    out = ctx.renormalize(dev(torch, U), [dev(torch, o) for o in ops], slices=S, ndiag=G)
    for i, (got, want) in enumerate(zip(out, oracle.renormalize(U, ops, S=S, G=G))):
        assert_bitexact(got.cpu().numpy(), want, "seed %d n=%d D=%d S=%d G=%d operator %d" % (seed, n, D, S, G, i))


def test_renormalize_fp64_and_errors(oz):
    ozaki, ctx, torch = oz
    n, D = 130, 33
    ops = wl.block_operators(n, 2, seed=10)
    U = np.linalg.qr(np.random.default_rng(11).standard_normal((n, D)))[0]
    out = ctx.renormalize(dev(torch, U), [dev(torch, o) for o in ops], slices=0)
    gam = n * U64 / (1 - n * U64)
    for O, got in zip(ops, out):
        bound = 3 * gam * (np.abs(U).T @ np.abs(O) @ np.abs(U))
        assert np.all(np.abs(got.cpu().numpy() - U.T @ O @ U) <= bound)
    with pytest.raises(ValueError):
        ctx.renormalize(dev(torch, U), [dev(torch, np.zeros((n, n + 1)))])
    with pytest.raises(ozaki.OzakiError):
        ctx.renormalize(dev(torch, np.zeros((n, n + 1))), [dev(torch, ops[0])])
    assert ctx.renormalize(dev(torch, U), [], slices=4) == []


@pytest.mark.parametrize("S", [0, 7])
def test_large_rdm(oz, S):
    """n = 2048 (a two-site tensor of D = 512, d = 4): the dominant quarter
    of the spectrum against the planted values."""
    t = wl.two_site_psi(2048, seed=12)
    A = t.psi @ t.psi.T
    w, Z, info = solve(oz, A, S, nev=512)
    assert info.status in (1, 2, 3), info.status
    assert np.max(np.abs(w - t.schmidt[:512] ** 2)) <= 64 * np.sqrt(2048) * u_eff(S) * w[0]
    res = np.linalg.norm(A @ Z - Z * w, axis=0)
    assert np.max(res) <= 64 * np.sqrt(2048) * u_eff(S) * w[0]


@pytest.mark.parametrize("S", [0, 3, 7])
@pytest.mark.parametrize("n,D,count", [(1, 1, 3), (40, 33, 5), (130, 64, 17), (300, 257, 3)])
def test_renormalize_batches(oz, S, n, D, count):
    """Several operators at once: counts below, at and past a batch, an odd one
    left over, the workspace of the per-operator query (batches of one), of the
    batch query and between; every form gives the bits of the two ozaki_dgemm
    calls per operator when emulated, and stays within the FP64 bound."""
    import ctypes
    ozaki, ctx, torch = oz
    ops = wl.block_operators(n, count, seed=n)
    U = np.linalg.qr(np.random.default_rng(n + D).standard_normal((n, D)))[0]
    dU, dops = dev(torch, U), [dev(torch, o) for o in ops]
    one = int(ozaki._lib.ozaki_renormalize_workspace_bytes(n, D, S, 0))
    many = int(ozaki._lib.ozaki_renormalize_batch_bytes(n, D, count, S, 0))
    assert many >= one
    want = oracle.renormalize(U, ops, S=S) if S else None
    gam = (n + 1) * U64 / (1 - (n + 1) * U64)
    for size in sorted({one, (one + many) // 2, many, many + 4096}):
        ws = torch.empty(max(size, 1), dtype=torch.uint8, device="cuda")
        out = ctx.renormalize(dU, dops, slices=S, workspace=ws)
        for k, got in enumerate(out):
            if S:
                assert_bitexact(got.cpu().numpy(), want[k], "operator %d, %d bytes" % (k, size))
            else:
                bound = 3 * gam * (np.abs(U).T @ np.abs(ops[k]) @ np.abs(U))
                assert np.all(np.abs(got.cpu().numpy() - U.T @ ops[k] @ U) <= bound)
    with pytest.raises(ozaki.OzakiError):
        ctx.renormalize(dU, dops, slices=S, workspace=torch.empty(max(one - 256, 0) or 1, dtype=torch.uint8,
                                                                  device="cuda")[: max(one - 256, 0)])
    if n == D:
        return
    # an output over the next operator: one by one, in order
    big = torch.zeros(2, n, n, dtype=torch.float64, device="cuda")
    big[0], big[1] = dops[0], dops[1]
    ctx.renormalize(dU, [big[0], big[1]], slices=S,
                    outs=[torch.empty(D, n, dtype=torch.float64, device="cuda")[:, :D], big[0][:D, :D]])
    ref = ctx.renormalize(dU, [dops[1]], slices=S)[0]
    assert torch.equal(big[0][:D, :D], ref)


@pytest.mark.parametrize("n", [320, 513])
@pytest.mark.parametrize("nev", ["all", "quarter"])
def test_clustered_eigenvalues_do_not_drift(oz, n, nev):
    """Native FP64 on clusters of nearly equal eigenvalues, whose rows keep
    rotating by small angles for many sweeps: every eigenvalue within the
    rounding of a quotient w A w^T (two sums of length n) and of LAPACK's, 8
    sqrt(n) u |A|_2 each, and the residuals with it."""
    rng = np.random.default_rng(n)
    lam = np.repeat([4.0, 3.0, 2.0, 1.0], -(-n // 4))[:n] + 1e-9 * rng.standard_normal(n)
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    A = (Q * lam) @ Q.T
    A = 0.5 * (A + A.T)
    k = n if nev == "all" else n // 4
    w, Z, info = solve(oz, A, nev=k)
    assert info.status == 1
    bound = 16 * np.sqrt(n) * U64 * 4.0
    assert np.max(np.abs(w - np.linalg.eigvalsh(A)[::-1][:k])) <= bound
    assert np.all(np.diff(w) <= 0)
    assert abs(info.trace - np.trace(A)) <= n * bound


@pytest.mark.parametrize("n", [65, 200, 513])
@pytest.mark.parametrize("kind", ["flat", "clusters", "graded"])
@pytest.mark.parametrize("tol", [1e-4, 1e-7])
def test_tolerance_of_the_caller(oz, n, kind, tol):
    """What a solve with a tolerance of its own leaves between the eigenvectors:
    at most the 0.1 tol |A|_F below which a sweep rotates nothing, and twice
    that where the second sweep that meets nothing above tol ends it."""
    rng = np.random.default_rng(n)
    lam = {"flat": np.linspace(2.0, 1.0, n), "graded": np.exp(-np.arange(n) / (n / 64.0)),
           "clusters": np.repeat([4.0, 3.0, 2.0, 1.0], -(-n // 4))[:n] + 1e-9 * rng.standard_normal(n)}[kind]
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    A = (Q * lam) @ Q.T
    A = 0.5 * (A + A.T)
    w, Z, info = solve(oz, A, tol=tol)
    assert info.status == 1 and info.off <= tol
    M = Z.T @ A @ Z
    assert np.max(np.abs(M - np.diag(np.diag(M)))) <= 0.2 * tol * np.linalg.norm(A)


@pytest.mark.parametrize("S", [0, 6])
@pytest.mark.parametrize("how", ["default", "tuned", "named"])
def test_renormalize_batches_on_every_context(oz, S, how):
    """Contexts that were tuned, or whose caller named a tile variant, work on
    several operators at once like any other (phase timing records a pass over
    a batch each: fewer records than operators), with the same bits."""
    ozaki, ctx, torch = oz
    n, D, count = 300, 130, 5
    ops = wl.block_operators(n, count, seed=7)
    U = np.linalg.qr(np.random.default_rng(3).standard_normal((n, D)))[0]
    dU, dops = dev(torch, U), [dev(torch, o) for o in ops]
    variants = [v for v, _, _ in ozaki.pair_variants(6)] if how == "named" and S else [None]
    want = ctx.renormalize(dU, dops, slices=S)
    if S:
        for got, ref in zip(want, oracle.renormalize(U, ops, S=S)):
            assert_bitexact(got.cpu().numpy(), ref)
    try:
        if how == "tuned":
            ctx.tune(dops[0], dU, slices=6)
        for v in variants:
            if v is not None:
                ctx.set_variant(6, 0, v)
            ctx.set_timing(True)
            ctx.phase_times()
            out = ctx.renormalize(dU, dops, slices=S)
            rec = ctx.phase_times()
            ctx.set_timing(False)
            assert len(rec) == (5 if S else 2), rec
            assert [r for r in rec if r[1] < 0] == []
            for a, b in zip(out, want):
                assert torch.equal(a, b)
    finally:
        ctx.set_timing(False)
        ctx.set_variant(6, 0, -1)


@pytest.mark.parametrize("S", [0, 7])
def test_renormalize_without_memory_for_a_batch(oz, S, monkeypatch):
    """Where the batch's workspace cannot be had, the call takes the
    per-operator one; results are the same."""
    ozaki, ctx, torch = oz
    n, D, count = 260, 40, 6
    ops = [dev(torch, o) for o in wl.block_operators(n, count, seed=11)]
    U = dev(torch, np.linalg.qr(np.random.default_rng(11).standard_normal((n, D)))[0])
    want = ctx.renormalize(U, ops, slices=S)
    one = int(ozaki._lib.ozaki_renormalize_workspace_bytes(n, D, S, 0))
    assert ozaki._lib.ozaki_renormalize_batch_bytes(n, D, count, S, 0) > one
    empty, asked = torch.empty, []

    def scarce(*size, **kw):
        if kw.get("dtype") is torch.uint8:
            asked.append(size[0])
            if size[0] > one:
                raise torch.cuda.OutOfMemoryError("no memory for the batch")
        return empty(*size, **kw)

    monkeypatch.setattr(ozaki.torch, "empty", scarce)
    out = ctx.renormalize(U, ops, slices=S)
    assert len(asked) == 2 and asked[1] == one
    for a, b in zip(out, want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("S", [0, 6])
@pytest.mark.parametrize("n", [65, 128, 129, 320])
@pytest.mark.parametrize("kind,steps", [("graded", 2), ("goe", 2), ("diagonal", 0), ("singular_first", 0),
                                        ("singular_second", 1)])
def test_qr_iteration_steps(oz, S, n, kind, steps):
    """How many steps of QR iteration the sweeps start from: both on a graded
    and on a random spectrum, none on a diagonal matrix; none where half of the
    eigenvalues sit at minus the first step's shift (3e-7 |A|_F: M + mu I is
    singular) and one where they sit at minus the second's (3e-12 |A|_F, which
    the first step still takes).  Each converges, and on the graded spectrum in
    ten sweeps at most where the matrix itself takes 15 to 29.  (Emulated sweeps
    that start from the matrix itself, half of its values one cluster, are left
    out of the accuracy check: their rounding gathers over 34 sweeps, to 1.2
    times the bound on residuals at n = 320, S = 6, and to 2.3 times over 39
    where no solve starts from QR iteration.)"""
    ozaki, ctx, torch = oz
    rng = np.random.default_rng(n)
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    lam = rng.uniform(0.5, 1.0, n)
    if kind == "graded":
        lam = np.exp(-np.arange(n) / (n / 64.0))
    elif kind == "goe":
        lam = rng.standard_normal(n)
    elif kind != "diagonal":
        lam[: n // 2] = -(3e-7 if kind == "singular_first" else 3e-12) * np.linalg.norm(lam[n // 2:])
    A = np.diag(lam) if kind == "diagonal" else (Q * lam) @ Q.T
    A = 0.5 * (A + A.T)
    nev = n // 4 if kind == "graded" else n
    eig = ozaki.RdmEig(ctx, n, S)
    try:
        # (from the matrix itself, half of its values one cluster: up to 39 sweeps at n = 320, S = 6)
        w, Z, info = eig.solve(dev(torch, A), nev, max_sweeps=60)
        assert eig.start_steps == steps
        assert info.status == 1
        if S == 0 or kind != "singular_first":
            check_eigenpairs(A, w.cpu().numpy(), Z.cpu().numpy(), S)
        if kind == "graded":
            assert info.sweeps <= 10
        # of the last solve: a diagonal matrix next, on the same plan
        eig.solve(dev(torch, np.diag(np.arange(n) + 1.0)), nev)
        assert eig.start_steps == 0
    finally:
        eig.close()


@pytest.mark.parametrize("n,D,count", [(1025, 321, 5), (700, 255, 16), (4095, 255, 16)])
def test_renormalize_native_batches_on_tiles(oz, n, D, count):
    """Native batches of more 64 x 64 tiles than the split kernel takes, odd
    extents: both products on 64 x 64 tiles, and (16 operators of n = 4095) the
    first on 128 x 128; within the FP64 bound of the two products."""
    ozaki, ctx, torch = oz
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    ops = [torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64) for _ in range(count)]
    U = torch.linalg.qr(torch.randn(n, D, generator=g, device="cuda", dtype=torch.float64))[0].contiguous()
    out = ctx.renormalize(U, ops, slices=0)
    gam = (n + 1) * U64 / (1 - (n + 1) * U64)
    aU = U.abs()
    aUt, Ut = aU.T.contiguous(), U.T.contiguous()
    for o, got in zip(ops, out):
        bound = 3 * gam * (aUt @ (o.abs() @ aU))
        assert bool(((got - Ut @ (o @ U)).abs() <= bound).all())


@pytest.mark.parametrize("n", [320, 513, 640])
def test_clustered_couplings_do_not_drift(oz, n):
    """Native FP64 on clusters of nearly equal eigenvalues: what a solve leaves
    between its eigenvectors is what it says of its own matrix, 0.1 tol |A|_F
    with the default tol = 4 sqrt(n_p) u, up to the rounding of A's products
    with the vectors (4 sqrt(n) u |A|_2)."""
    rng = np.random.default_rng(n + 1)
    lam = np.repeat([4.0, 3.0, 2.0, 1.0], -(-n // 4))[:n] + 1e-9 * rng.standard_normal(n)
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    A = (Q * lam) @ Q.T
    A = 0.5 * (A + A.T)
    w, Z, info = solve(oz, A)
    assert info.status == 1
    tol = 4 * np.sqrt(-(-n // 64) * 64) * U64
    M = Z.T @ A @ Z
    left = np.max(np.abs(M - np.diag(np.diag(M))))
    assert left <= 0.1 * tol * np.linalg.norm(A) + 4 * np.sqrt(n) * U64 * 4.0, left / (tol * np.linalg.norm(A))
