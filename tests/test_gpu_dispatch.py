"""The kernels' dispatch rules at their edges, on small systems with a known answer.

Systems: block-tridiagonal SPD matrices of 3x3 blocks with a dominant diagonal (condition
number below 4), so that a solve to 1e-13 leaves an error below 4e-13 plus the rounding of
the products, and 1e-11 is asked.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2111_09294_amd as D  # noqa: E402

DEV = "cuda:0"


def chain(nb, seed=0):
    """K (scipy CSR) of nb block rows: 3x3 blocks on three block diagonals."""
    import scipy.sparse as sp
    rng = np.random.default_rng(seed)
    off = rng.uniform(-0.1, 0.1, (max(nb - 1, 0), 3, 3))
    diag = rng.uniform(-0.05, 0.05, (nb, 3, 3))
    diag = 0.5 * (diag + diag.transpose(0, 2, 1)) + 1.5 * np.eye(3)
    rows = np.arange(nb)
    blocks = np.concatenate([diag, off, off.transpose(0, 2, 1)])
    I = np.concatenate([rows, rows[:-1], rows[1:]])
    J = np.concatenate([rows, rows[1:], rows[:-1]])
    r = (3 * I[:, None, None] + np.arange(3)[None, :, None]) + np.zeros((1, 1, 3), int)
    c = (3 * J[:, None, None] + np.arange(3)[None, None, :]) + np.zeros((1, 3, 1), int)
    K = sp.csr_matrix((blocks.reshape(-1), (r.reshape(-1), c.reshape(-1))), shape=(3 * nb, 3 * nb))
    K.sort_indices()
    return K


def solver(K, sel, block=3):
    """Solver with nodal blocks of `block` unknowns and Z = unit vectors of the unknowns sel."""
    n, k = K.shape[0], len(sel)
    zp = np.zeros(n + 1, np.int64)
    zp[np.asarray(sel, int) + 1] = 1
    t = lambda a, dt: torch.as_tensor(np.ascontiguousarray(a), device=DEV).to(dt)  # noqa: E731
    bp = np.unique(np.concatenate([np.arange(0, n, block), [n]]))
    return D.Solver(n, t(K.indptr, torch.int64), t(K.indices, torch.int32), t(K.data, torch.float64), k,
                    t(np.cumsum(zp), torch.int64), t(np.arange(k), torch.int32),
                    t(np.ones(k), torch.float64), t(bp, torch.int32))


@pytest.mark.parametrize("k", [1, 2, 63, 64, 65, 127, 1023, 1024, 1025])
def test_coarse_product_forms(k):
    """E^-1 g by rows (k <= 1024) and by tiles; E = K at every third-or-so unknown."""
    K = chain(700)
    sel = np.sort(np.random.default_rng(k).permutation(2100)[:k])
    g = np.random.default_rng(1).standard_normal(k)
    with solver(K, sel) as s:
        d = s.coarse_apply(torch.as_tensor(g, device=DEV)).cpu().numpy()
        # the whole iteration on the same form
        x = np.random.default_rng(2).standard_normal(2100)
        u, info = s.solve(torch.as_tensor(K @ x, device=DEV), tol=1e-13)
    ref = np.linalg.solve(K[sel][:, sel].toarray(), g)
    assert np.linalg.norm(d - ref) <= 1e-13 * k ** 0.5 * np.linalg.norm(ref) + 1e-14
    assert info["status"] == 0
    assert np.linalg.norm(u.cpu().numpy() - x) <= 1e-11 * np.linalg.norm(x)


@pytest.mark.parametrize("cond", [1e3, 1e6, 1e9])
def test_pivot_inverse_accuracy(cond):
    """The inverse of one 64 x 64 pivot block: elimination of one pivot after the other leaves
    |I - S P| at 0.8 eps cond in a model with these spectra, products with explicit inverses of
    16 x 16 blocks 5 to 22 eps cond from condition 1e6 on; the line is drawn at 4."""
    import scipy.sparse as sp
    rng = np.random.default_rng(5)
    Q = np.linalg.qr(rng.standard_normal((64, 64)))[0]
    S = Q * rng.permutation(np.logspace(0, -np.log10(cond), 64)) @ Q.T
    d = 1 / np.sqrt(np.diag(S))
    S = S * d * d[:, None]
    S = 0.5 * (S + S.T)
    K = sp.block_diag([S, sp.identity(2)]).tocsr()
    K.sort_indices()
    with solver(K, np.arange(64)) as s:
        P = np.stack([s.coarse_apply(torch.as_tensor(e, device=DEV)).cpu().numpy() for e in np.eye(64)], 1)
    assert np.linalg.norm(np.eye(64) - S @ P) <= 4 * np.finfo(float).eps * max(np.linalg.cond(S), 64)


@pytest.mark.parametrize("nb", [1, 85, 86, 4096, 4097, 32768, 32769, 131072, 131073, 294912, 294913])
def test_step_length_partials(nb):
    """p^T q from up to 64 partials, from the SpMV's own up to 4608 (64 block rows each; in
    rounds of at most 512, 2048 and 4608), and through a first stage above; 85 block rows
    fill one tile of the update, 86 start another.  Blocks of 6 unknowns, the last one of 3
    where nb is odd."""
    K = chain(nb)
    x = np.random.default_rng(3).standard_normal(3 * nb)
    with solver(K, [0] if nb > 1 else [], block=6) as s:
        u, info = s.solve(torch.as_tensor(K @ x, device=DEV), tol=1e-13)
    assert info["status"] == 0
    assert np.linalg.norm(u.cpu().numpy() - x) <= 1e-11 * np.linalg.norm(x)


@pytest.mark.parametrize("nb", [4162, 294912])
def test_breakdown_keeps_the_last_iterate(nb):
    """A breakdown of the second step with p^T q summed by the update (66 and 4608 partials):
    u stays what one iteration made it, bit for bit and every time, alone and among other
    systems.  K is block diagonal in pairs [[A, 2A], [2A, A]], M^-1 K has the eigenvalues 3
    and -1 only, so from f in both eigenspaces (f^T M^-1 K M^-1 f > 0) the second direction's
    p^T K p is negative."""
    import scipy.sparse as sp
    A = np.array([[4.0, 1.0, 0.5], [1.0, 3.0, 0.2], [0.5, 0.2, 2.0]])
    K = sp.kron(sp.identity(nb // 2), np.block([[A, 2 * A], [2 * A, A]])).tocsr()
    K.sort_indices()
    x = np.random.default_rng(6).uniform(0.5, 1.5, (nb // 2, 3)) @ A
    f = torch.as_tensor(np.concatenate([2 * x, 0 * x], 1).reshape(-1), device=DEV)
    C = chain(700)
    y = np.random.default_rng(7).standard_normal(2100)
    g = torch.as_tensor(C @ y, device=DEV)
    with solver(K, []) as s, solver(C, [0]) as healthy, solver(K, []) as other:
        one, ref = s.solve(f, tol=1e-13, max_iter=1, raise_on_error=False)
        assert ref["status"] == D.abi.NOT_CONVERGED and ref["iterations"] == 1
        for _ in range(3):
            u, info = s.solve(f, tol=1e-13, raise_on_error=False)
            assert info["status"] == D.abi.EBREAKDOWN and info["bad_index"] == 1 and info["iterations"] == 1
            assert torch.equal(u, one) and info["rel_res_true"] == ref["rel_res_true"]
            us, infos = D.solve_many([healthy, s, other], [g, f, f], tol=1e-13, raise_on_error=False)
            assert [i["status"] for i in infos] == [0, D.abi.EBREAKDOWN, D.abi.EBREAKDOWN]
            assert torch.equal(us[1], one) and torch.equal(us[2], one)
            assert np.linalg.norm(us[0].cpu().numpy() - y) <= 1e-11 * np.linalg.norm(y)


@pytest.mark.parametrize("sizes", [[19, 31, 32, 33, 5], [63, 64, 65, 12], [96, 97, 128, 129], [255, 256, 257, 3, 18],
                                   [513, 24, 1000]])
def test_dense_block_tiles(sizes):
    """Subdomain-sized blocks at the edges of the inverse's tiles (32), of the sweeps' (64) and
    of the apply's strips (8 tiles), beside nodal blocks, each against LAPACK."""
    n = -(-sum(sizes) // 3) * 3
    K = chain(n // 3, seed=7)
    bp = np.cumsum([0] + sizes + ([n - sum(sizes)] if n > sum(sizes) else []))
    r = np.random.default_rng(8).standard_normal(n)
    t = lambda a, dt: torch.as_tensor(np.ascontiguousarray(a), device=DEV).to(dt)  # noqa: E731
    with D.Solver(n, t(K.indptr, torch.int64), t(K.indices, torch.int32), t(K.data, torch.float64), 0, None, None,
                  None, t(bp, torch.int32)) as s:
        y = s.bj_apply(t(r, torch.float64)).cpu().numpy()
        y32 = s.bj_apply_fp32(t(r, torch.float64)).cpu().numpy()
        u, info = s.solve(t(K @ r, torch.float64), tol=1e-13)
    assert info["status"] == 0 and np.linalg.norm(u.cpu().numpy() - r) <= 1e-11 * np.linalg.norm(r)
    for a, b in zip(bp[:-1], bp[1:]):
        Minv = np.linalg.inv(K[a:b, a:b].toarray())
        ref = Minv @ r[a:b]
        assert np.linalg.norm(y[a:b] - ref) <= (b - a) * 4e-15 * np.linalg.norm(ref)
        bound = 2.0 ** -24 * np.abs(Minv) @ np.abs(r[a:b])
        assert np.all(np.abs(y32[a:b] - ref) <= 1.01 * bound + (b - a) * 4e-15 * np.abs(ref).max())


@pytest.mark.parametrize("nb, long", [(40, 30), (1500, 64), (20000, 300), (120000, 300)])
def test_few_long_rows(nb, long):
    """Two block rows far longer than the rest, which set the SpMV's lanes per row: the product
    entry by entry (two sums of at most m products differ by 2 m eps (|K| |x|)), and alone and
    among other systems the same iterates, bit for bit."""
    import scipy.sparse as sp
    rng = np.random.default_rng(30)
    K = chain(nb)
    rows = 3 * rng.choice(nb, 2, replace=False)
    I, J = np.repeat(rows, long), 3 * np.concatenate([rng.choice(nb, long, replace=False) for _ in rows])
    C = sp.csr_matrix((np.full(len(I), 0.3 / long), (I, J)), shape=K.shape)
    K = (K + C + C.T).tocsr()
    K.sort_indices()
    x = rng.standard_normal(3 * nb)
    f = torch.as_tensor(K @ x, device=DEV)
    m = int(np.diff(K.indptr).max())
    with solver(K, [0, 5]) as s, solver(chain(7), []) as other:
        y = s.spmv(torch.as_tensor(x, device=DEV)).cpu().numpy()
        assert np.all(np.abs(y - K @ x) <= 2 * m * np.finfo(float).eps * (abs(K) @ np.abs(x)))
        u, info = s.solve(f, tol=1e-13)
        us, _ = D.solve_many([other, s], [torch.ones(21, dtype=torch.float64, device=DEV), f], tol=1e-13)
        assert info["status"] == 0 and torch.equal(us[1], u)
    assert np.linalg.norm(u.cpu().numpy() - x) <= 1e-11 * np.linalg.norm(x)


@pytest.mark.parametrize("seed", [0, 1])
def test_many_small_dense_blocks(seed):
    """Blocks of 19 to 130 unknowns, every size twice in a mixed order, each against LAPACK."""
    rng = np.random.default_rng(20 + seed)
    sizes = rng.permutation(np.repeat(np.arange(19, 131), 2))
    n = -(-int(sizes.sum()) // 3) * 3
    K = chain(n // 3, seed=21 + seed)
    d = 10.0 ** rng.uniform(-3, 3, n)  # rows of unequal scale
    import scipy.sparse as sp
    K = (sp.diags(d) @ K @ sp.diags(d)).tocsr()
    K = (0.5 * (K + K.T)).tocsr()
    K.sort_indices()
    bp = np.concatenate([[0], np.cumsum(sizes)])
    bp = np.concatenate([bp, [n]]) if n > bp[-1] else bp
    r = rng.standard_normal(n) * d
    t = lambda a, dt: torch.as_tensor(np.ascontiguousarray(a), device=DEV).to(dt)  # noqa: E731
    with D.Solver(n, t(K.indptr, torch.int64), t(K.indices, torch.int32), t(K.data, torch.float64), 0, None, None,
                  None, t(bp, torch.int32)) as s:
        y = s.bj_apply(t(r, torch.float64)).cpu().numpy()
    for a, b in zip(bp[:-1], bp[1:]):
        ref = np.linalg.solve(K[a:b, a:b].toarray() / d[a:b, None] / d[None, a:b], r[a:b] / d[a:b])
        assert np.linalg.norm(y[a:b] * d[a:b] - ref) <= (b - a) * 4e-15 * np.linalg.norm(ref), (a, b)


@pytest.mark.parametrize("size, bad", [(19, 0), (40, 39), (64, 17), (65, 64), (100, 30), (128, 127), (129, 128)])
def test_small_dense_block_that_is_not_spd(size, bad):
    """A negative diagonal entry, in the first and in the second tile: the block's index."""
    n = 4 * 3 * size
    K = chain(n // 3, seed=22).tolil()
    K[2 * size + bad, 2 * size + bad] = -1.0
    K = K.tocsr()
    K.sort_indices()
    t = lambda a, dt: torch.as_tensor(np.ascontiguousarray(a), device=DEV).to(dt)  # noqa: E731
    with pytest.raises(D.DpcgError) as e:
        D.Solver(n, t(K.indptr, torch.int64), t(K.indices, torch.int32), t(K.data, torch.float64), 0, None, None,
                 None, t(np.arange(0, n + 1, size), torch.int32))
    assert e.value.code == D.abi.EBLOCK_NOT_SPD and e.value.info.bad_index == 2


@pytest.mark.parametrize("nbs", [[1, 170, 171, 86], [1365, 1366, 2730, 2731], [20000, 87382, 5], [174762, 174763]])
def test_many_prolongation_grid(nbs):
    """Several systems at the edges of the prolongation's grid (512 rows per workgroup, from
    eight workgroups on a multiple of eight): the single solves' iterates, bit for bit."""
    Ks = [chain(nb, seed=i) for i, nb in enumerate(nbs)]
    xs = [np.random.default_rng(11 + i).standard_normal(3 * nb) for i, nb in enumerate(nbs)]
    fs = [torch.as_tensor(K @ x, device=DEV) for K, x in zip(Ks, xs)]
    ss = [solver(K, np.arange(0, 3 * nb, 97) if nb > 1 else []) for K, nb in zip(Ks, nbs)]
    try:
        us, infos = D.solve_many(ss, fs, tol=1e-13)
        for s, f, u, x, i in zip(ss, fs, us, xs, infos):
            one, ref = s.solve(f, tol=1e-13)
            assert i["status"] == 0 and i["iterations"] == ref["iterations"] and torch.equal(u, one)
            assert np.linalg.norm(u.cpu().numpy() - x) <= 1e-11 * np.linalg.norm(x)
    finally:
        for s in ss:
            s.close()


def inverse_errors(m, decades, count, seed):
    """Relative errors of M^-1 r for blocks of m unknowns with spectra spread evenly over the decades."""
    import scipy.sparse as sp
    rng = np.random.default_rng(seed)
    blocks = []
    for _ in range(count):
        Q = np.linalg.qr(rng.standard_normal((m, m)))[0]
        S = Q * np.logspace(0, -decades, m) @ Q.T
        blocks.append(0.5 * (S + S.T))
    n = 3 * m * (-(-count // 3))
    K = sp.block_diag(blocks + [sp.identity(n - m * count)] * (n > m * count)).tocsr()
    K.sort_indices()
    r = rng.standard_normal(n)
    t = lambda a, dt: torch.as_tensor(np.ascontiguousarray(a), device=DEV).to(dt)  # noqa: E731
    bp = np.unique(np.concatenate([np.arange(0, m * count + 1, m), [n]]))
    with D.Solver(n, t(K.indptr, torch.int64), t(K.indices, torch.int32), t(K.data, torch.float64), 0, None,
                  None, None, t(bp, torch.int32)) as s:
        y = s.bj_apply(t(r, torch.float64)).cpu().numpy()
    errs = []
    for i, S in enumerate(blocks):
        rb = r[i * m:(i + 1) * m]
        x = np.linalg.solve(S, rb).astype(np.longdouble)
        for _ in range(4):  # refined in extended precision
            x = x + np.linalg.solve(S, (rb - S.astype(np.longdouble) @ x).astype(float))
        errs.append(float(np.linalg.norm(y[i * m:(i + 1) * m] - x) / np.linalg.norm(x)))
    return errs


@pytest.mark.parametrize("m", [48, 80, 96, 129, 160, 400])
def test_dense_inverse_accuracy(m):
    """Condition 1e6: a backward stable inverse leaves a forward error of a modest multiple of
    eps cond; the line is drawn at one.  (Rows by an explicit pivot inverse, unrefined, leave
    up to eps cond^2: 50 eps cond at 80.)"""
    assert max(inverse_errors(m, 6, 3, 40 + m)) <= np.finfo(float).eps * 1e6


def test_dense_inverse_roundings():
    """An entry is rounded at its own magnitude once per pair of pivot tiles: between 2 pairs
    (129 unknowns) and 7 (800) the error grows by sqrt(7 / 2) = 1.9 at most (tripled where every
    product of a pair was added to the entry by itself)."""
    small, large = (np.mean(inverse_errors(m, 2, 3, 50 + m)) for m in (129, 800))
    assert large <= 1.9 * small


@pytest.mark.parametrize("sizes", [[129, 64], [192, 193], [257, 320, 500]])
def test_dense_inverses_repeat(sizes):
    """Blocks of two to eight tiles of the sweeps, set up again: the same inverses, bit for bit."""
    n = -(-sum(sizes) // 3) * 3
    K = chain(n // 3, seed=9)
    bp = np.cumsum([0] + sizes + ([n - sum(sizes)] if n > sum(sizes) else []))
    t = lambda a, dt: torch.as_tensor(np.ascontiguousarray(a), device=DEV).to(dt)  # noqa: E731
    r = t(np.random.default_rng(10).standard_normal(n), torch.float64)
    ys = []
    for _ in range(4):
        with D.Solver(n, t(K.indptr, torch.int64), t(K.indices, torch.int32), t(K.data, torch.float64), 0, None,
                      None, None, t(bp, torch.int32)) as s:
            ys.append(s.bj_apply(r))
    assert all(torch.equal(y, ys[0]) for y in ys[1:])


@pytest.mark.parametrize("nrhs", [1, 7, 8, 9, 16, 17, 32])
def test_batch_widths(problems, nrhs):
    """The batch layout's widths (8, 16, 32 columns): K X of an enriched mesh entry by entry
    (pairs, twin rows and long rows; two sums of at most m products differ by 2 m eps
    (|K| |x|)), and a solve with known columns, unequal in length to finish apart."""
    p = problems("edge10")
    K = p.K_scipy().tocsr()
    X = np.random.default_rng(nrhs).standard_normal((p.n, nrhs))
    with D.Solver.from_problem(p, DEV) as s:
        Y = s.spmv_batch(torch.as_tensor(X, device=DEV)).cpu().numpy()
    m = int(np.diff(K.indptr).max())
    assert np.all(np.abs(Y - K @ X) <= 2 * m * np.finfo(float).eps * (abs(K) @ np.abs(X)))
    nb = 1001
    C = chain(nb, seed=2)
    X = np.random.default_rng(nrhs).standard_normal((3 * nb, nrhs)) * 10.0 ** np.arange(nrhs)[None, :]
    X[: 3 * (nb // 2), -1] = 0.0
    with solver(C, np.arange(0, 3 * nb, 50)) as s:
        U, infos = s.solve_batch(torch.as_tensor(C @ X, device=DEV), tol=1e-13)
    err = np.linalg.norm(U.cpu().numpy() - X, axis=0)
    assert all(i["status"] == 0 for i in infos) and np.all(err <= 1e-11 * np.linalg.norm(X, axis=0))


def test_kept_entries_of_kz(problems):
    """(K Z)^T without the entries that are only rounding: g = Z^T a - (K Z)^T b against scipy
    within the rounding of the sums, fewer stored than structural entries, and another set after
    a values update (springs to the ground make K Z dense, without them it is sparse again), in
    single and batched solves of the same handle."""
    p = problems("penny12")
    K, Z = p.K_scipy().tocsr(), p.Z_scipy().tocsr()
    G = K.copy()
    G.setdiag(1.1 * K.diagonal())
    t = lambda a, dt: torch.as_tensor(np.ascontiguousarray(a), device=DEV).to(dt)  # noqa: E731
    rng = np.random.default_rng(5)
    a, b, X = rng.standard_normal(p.n), rng.standard_normal(p.n), rng.standard_normal((p.n, 5))
    kept = []
    with D.Solver.from_problem(p, DEV) as s:
        for M in (K, G, K):
            s.update_values(t(M.indptr, torch.int64), t(M.indices, torch.int32), t(M.data, torch.float64))
            kept.append(s.stats()["nnz_kz"])
            g = s.restrict(t(a, torch.float64), t(b, torch.float64)).cpu().numpy()
            scale = abs(Z).T @ np.abs(a) + abs(Z).T @ (abs(M) @ np.abs(b))
            assert np.all(np.abs(g - (Z.T @ a - Z.T @ (M @ b))) <= 1e-13 * scale)
            U, infos = s.solve_batch(t(M @ X, torch.float64), tol=1e-12)
            for j in range(X.shape[1]):
                u, info = s.solve(t((M @ X)[:, j], torch.float64), tol=1e-12)
                assert info["status"] == 0 and infos[j]["status"] == 0
                assert torch.linalg.norm(U[:, j] - u) <= 1e-8 * torch.linalg.norm(u)
    assert kept[0] == kept[2] < 0.9 * kept[1]


def test_small_entries_of_kz_are_kept():
    """Entries of K Z far below (sum |K|) (max |z|) of their row, but not below the rounding of
    their own sum: rows of tiny couplings and tiny components beside large ones.  Each g is one
    product of two entries or a sum of two, without cancellation: 4 eps."""
    import scipy.sparse as sp
    rng = np.random.default_rng(12)
    nb = 40
    K = sp.lil_matrix((3 * nb, 3 * nb))
    K.setdiag(rng.uniform(1.0, 2.0, 3 * nb))
    for d in range(0, 60, 3):  # triplet d couples to its partner by 1e-20
        K[d, d + 60] = K[d + 60, d] = 1e-20 * rng.uniform(1.0, 2.0)
    K = K.tocsr()
    K.sort_indices()
    Z = np.zeros((3 * nb, 2))
    Z[:60, 0] = 1e-18 * rng.uniform(1.0, 2.0, 60)  # tiny beside its partner's
    Z[60:, 0] = rng.uniform(1.0, 2.0, 60)
    Z[60:, 1] = rng.uniform(1.0, 2.0, 60)          # reaches the first half by the couplings only
    Zs = sp.csr_matrix(Z)
    t = lambda a, dt: torch.as_tensor(np.ascontiguousarray(a), device=DEV).to(dt)  # noqa: E731
    zero, KZ = torch.zeros(3 * nb, dtype=torch.float64, device=DEV), K @ Z
    with D.Solver(3 * nb, t(K.indptr, torch.int64), t(K.indices, torch.int32), t(K.data, torch.float64), 2,
                  t(Zs.indptr, torch.int64), t(Zs.indices, torch.int32), t(Zs.data, torch.float64),
                  t(np.arange(0, 3 * nb + 1, 3), torch.int32)) as s:
        for d in range(0, 3 * nb, 7):
            b = zero.clone()
            b[d] = 1.0
            g = s.restrict(zero, b).cpu().numpy()
            assert np.all(np.abs(g + KZ[d]) <= 4 * np.finfo(float).eps * np.abs(KZ[d])), (d, g, KZ[d])
