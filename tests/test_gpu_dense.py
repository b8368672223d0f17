"""Dense factor and solve kernels at the edges of their blocks, against FP64
host arithmetic.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def nb():
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    import paper_2606_24154_amd as nb
    return nb


def dev(a, dtype=torch.float64):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0", dtype=dtype)


def factors(n, seed):
    rng = np.random.default_rng(seed)
    L = np.tril(rng.uniform(-1, 1, (n, n)), -1) / np.sqrt(n)
    U = np.triu(rng.uniform(-1, 1, (n, n)), 1) / np.sqrt(n) + np.diag(rng.choice([-1.0, 1.0], n) * rng.uniform(1, 3, n))
    piv = np.array([rng.integers(k, n) for k in range(n)])
    return rng, L, U, piv


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 129, 700])
@pytest.mark.parametrize("nrhs", [1, 3, 4, 9])
def test_solves_from_factors(nb, n, nrhs):
    """X from given factors and interchanges.  Substitution leaves
    |P b - L U x| <= 3 n eps |L + I| |U| |x| (Higham, Accuracy and Stability, theorem
    9.4); twice that covers the residual's own rounding on the host."""
    rng, L, U, piv = factors(n, 100 * n + nrhs)
    B = rng.standard_normal((nrhs, n))
    LU, ipiv = dev((L + U).T), dev(piv, torch.int32)
    X = nb.solve_factored(LU, ipiv, dev(B)).cpu().numpy()
    PB = B.T.copy()
    for k in range(n):
        PB[[k, piv[k]]] = PB[[piv[k], k]]
    L1 = L + np.eye(n)
    bound = 6 * n * EPS * (np.abs(L1) @ (np.abs(U) @ np.abs(X.T)))
    assert (np.abs(PB - L1 @ (U @ X.T)) <= bound).all()
    # a column by itself, and in place: the same bits
    one = dev(B[-1])
    nb.solve_factored(LU, ipiv, one, sigma=one)
    assert np.array_equal(one.cpu().numpy(), X[-1])


@pytest.mark.parametrize("n", [1, 65, 200])
@pytest.mark.parametrize("nrhs", [2, 6, 7])
def test_columns_of_a_last_pass(nb, n, nrhs):
    """Two or three columns solved together have the bits of each by itself."""
    rng, L, U, piv = factors(n, 100 * n + nrhs)
    B = rng.standard_normal((nrhs, n))
    LU, ipiv = dev((L + U).T), dev(piv, torch.int32)
    X = nb.solve_factored(LU, ipiv, dev(B))
    for k in range(nrhs):
        assert torch.equal(nb.solve_factored(LU, ipiv, dev(B[k])), X[k]), k


def test_solves_beyond_the_reciprocals_range(nb):
    """Pivots whose reciprocals overflow or are zero divide as IEEE division
    does, and an infinite solution leaves those solved before it alone."""
    n = 70
    U = np.eye(n)
    U[:5, :5] = np.diag([2.0, 5e-324, 1e308, 0.0, 3.0])
    B = np.ones((1, n))
    B[0, 1] = 5e-324
    U[2, 69] = 1.0
    X = nb.solve_factored(dev(U.T), dev(np.arange(n), torch.int32), dev(B)).cpu().numpy()[0]
    assert X[4] == 1.0 / 3.0 and X[1] != X[1] and np.isinf(X[3])  # 0 x inf enters rows 0 .. 2
    assert (X[5:] == 1.0).all()


def factor(nb, A):
    """(LU, ipiv) of P A = L U, A a (n, n) float64 tensor on the GPU."""
    At = A.T.contiguous()
    _, ipiv, _ = nb.solve(At, torch.ones(len(A), dtype=torch.float64, device="cuda:0"))
    return At.T, ipiv


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 257, 700])
def test_pivots(nb, n):
    """The interchanges of partial pivoting as LAPACK finds them, and among
    equal candidates the first row: in the second matrix every column is all ties, and
    each value is a power of two, so that the factors are exact."""
    import scipy.linalg
    rng = np.random.default_rng(n)
    A = rng.standard_normal((n, n))
    LU, ipiv = factor(nb, dev(A))
    ref, piv = scipy.linalg.lu_factor(A)
    assert np.array_equal(ipiv.cpu().numpy(), piv)
    # both factorisations are backward stable; their difference is rounding times the
    # condition of the leading blocks, random ones here: 1e-16 n^2 times 1e3
    assert np.abs(LU.cpu().numpy() - ref).max() <= 1e-13 * max(n, 10) ** 2
    W = np.eye(n) - np.tril(np.ones((n, n)), -1)
    W[:, -1] = 1.0
    LU, ipiv = factor(nb, dev(W))
    assert np.array_equal(ipiv.cpu().numpy(), np.arange(n))
    ref = W.copy()
    ref[:, -1] = 2.0 ** np.arange(n)
    assert np.array_equal(LU.cpu().numpy(), ref)


def test_factor_large(nb):
    """Past 256 waves' rows a panel's workgroups own 256 rows each: n = 16384
    + 70 begins there and ends with one wave per workgroup."""
    n = 16384 + 70
    g = torch.Generator(device="cuda:0").manual_seed(5)
    A = torch.randn(n, n, dtype=torch.float64, device="cuda:0", generator=g)
    x = torch.randn(n, dtype=torch.float64, device="cuda:0", generator=g)
    b = A @ x
    At = A.T.contiguous()
    y, ipiv, _ = nb.solve(At, b)
    assert float(torch.tril(At.T, -1).abs().max()) <= 1.0
    # backward error of the refined solve: a few n eps of |A| |x|
    bound = 4 * n * EPS * (A.abs() @ y.abs())
    assert bool(((A @ y - b).abs() <= bound).all())
    p = ipiv.cpu().numpy()
    assert (p >= np.arange(n)).all() and (p < n).all()


@pytest.mark.parametrize("n, precision", [(33_100, 0), (65_700, 1)])
def test_factor_larger(nb, n, precision):
    """Thousands of workgroups for a panel's rows of U, and in FP32 panels of more than
    256 workgroups.  A is 3 sqrt(n) times a permutation plus
    normal entries, whose singular values end near 2 sqrt(n): |A^-1| <= 1.1 / sqrt(n),
    |A| <= 5.1 sqrt(n), and the pivot rows are the permutation's (elsewhere a column's
    entries stay some standard deviations, 3 sqrt(n) is hundreds).  So |x - y| is at most
    5.7 times |y| x (the refinement's 1e-10, or the FP64 solve's rounding)."""
    g = torch.Generator(device="cuda:0").manual_seed(6)
    At = torch.randn(n, n, dtype=torch.float64, device="cuda:0", generator=g)  # column-major A
    row = torch.randperm(n, device="cuda:0", generator=g)  # of each column's large entry
    At[torch.arange(n, device="cuda:0"), row] += 3 * n**0.5
    y = torch.randn(n, dtype=torch.float64, device="cuda:0", generator=g)
    b = At.T @ y
    x, ipiv, info = nb.solve(At, b, precision)
    assert info.rel_resid <= (1e-10 if precision else 1e-13)
    assert float((x - y).norm() / y.norm()) <= 5.7 * (1e-10 if precision else 1e-13)
    perm = np.arange(n)
    for k, p in enumerate(ipiv.cpu().numpy()):
        perm[[k, p]] = perm[[p, k]]
    assert np.array_equal(perm, row.cpu().numpy())


def assembly_geometry(kind):
    """1242 elements, conductor and dielectric rows, the last group ragged: one
    cell's copies as usual, on a skewed lattice with more copies one way, with
    reflections, and with one row of 41."""
    from synth import Images, gem_cell
    g = gem_cell(k=17, nr=2, n_images=5)
    im = g.images
    if kind == "skew":
        return g.with_images(Images(a1=im.a1, a2=im.a2 + 0.3 * im.a1, n1=2, n2=30))
    if kind == "mirror":
        return g.with_images(Images(a1=im.a1, a2=im.a2, n1=2, n2=3, mirror_mask=5,
                                    mirror_pos=np.array([-2e-4, 0.0, -1.5e-3]),
                                    mirror_parity=np.array([1, 1, -1], np.int32)))
    if kind == "line":
        return g.with_images(Images(a1=im.a1, a2=im.a2, n1=0, n2=20))
    return g


@pytest.mark.parametrize("kind", ["cell", "skew", "mirror", "line"])
def test_grouped_assembly(nb, kind):
    """The matrix with far copies by lattice sums against the closed forms
    throughout, which collocation points handed in by the caller take, and
    sampled rows against the oracle.  1e-11 of a row's largest entry, as every
    assembly here; entry by entry 1e-10 where all copies count with one sign (an
    expansion is truncated below 3e-12, the closed forms round at 1e-11)."""
    import oracle
    g = assembly_geometry(kind)
    dp = nb.DevicePanels.from_geometry(g, "cuda:0")
    A = nb.assemble(dp).cpu().numpy().T
    D = nb.assemble(dp, colloc=[dev(c) for c in g.centroids().T]).cpu().numpy().T
    rows = np.unique(np.concatenate([np.arange(0, g.n, 97), [63, 64, g.n - 1]]))
    ref = oracle.assemble_rows(g, rows)
    assert (np.abs(A[rows] - ref).max(axis=1) <= 1e-11 * np.abs(ref).max(axis=1)).all()
    assert (np.abs(A - D).max(axis=1) <= 1e-11 * np.abs(D).max(axis=1)).all()
    if kind != "mirror":
        c = g.bc == 0
        assert (np.abs(A[c] - D[c]) <= 1e-10 * np.abs(D[c])).all()


def test_grouped_assembly_in_random_order(nb):
    """Groups of elements from all over the cell, as wide as the lattice: no copy is far
    from any, and every entry is a closed form's, as in the direct assembly (1e-11 of a
    row's largest entry, and 1e-10 entry by entry for conductors, as above)."""
    g = assembly_geometry("cell")
    g = g.subset(np.random.default_rng(3).permutation(g.n))
    dp = nb.DevicePanels.from_geometry(g, "cuda:0")
    A = nb.assemble(dp).cpu().numpy().T
    D = nb.assemble(dp, colloc=[dev(c) for c in g.centroids().T]).cpu().numpy().T
    assert (np.abs(A - D).max(axis=1) <= 1e-11 * np.abs(D).max(axis=1)).all()
    c = g.bc == 0
    assert (np.abs(A[c] - D[c]) <= 1e-10 * np.abs(D[c])).all()
