"""The Dyson solve and its adjoint at the edges of the blocked LU: bases
around multiples of its 16-column panels, of a wave (64 rows), of a workgroup
(256 rows) and of its largest size (304; above it the unblocked kernels run),
matrices that need row exchanges, pivots that vanish at a panel's first, inner
and last column.  Reference: dense solves in numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -53


@pytest.fixture(scope="module")
def tdx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_01875_amd as m
    return m


@pytest.fixture(scope="module")
def ctx(tdx):
    c = tdx.Context(0)
    yield c
    c.close()


SIZES = [1, 2, 15, 16, 17, 31, 33, 47, 48, 49, 63, 64, 65, 97, 127, 128, 130, 161, 255, 256, 257,
         303, 304, 305]


@pytest.mark.parametrize("n", SIZES)
def test_solve_and_adjoint_match_dense_solves(tdx, ctx, n):
    import torch
    print("lu", n, flush=True)
    n_w = 3
    rng = np.random.default_rng(n)
    cn = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)  # noqa: E731
    A = cn(n_w, n, n)       # dense and unordered: most columns exchange rows
    K = cn(n, n) + 2 * np.eye(n)
    chi0 = (np.eye(n) - A) @ np.linalg.inv(K)
    A = np.eye(n) - chi0 @ K
    g0, cbar = n // 3, cn(n_w)
    e = np.zeros(n)
    e[g0] = 1.0
    x = np.linalg.solve(A, chi0[:, :, g0:g0 + 1])[:, :, 0]
    a = np.linalg.solve(A.transpose(0, 2, 1), np.broadcast_to(e[:, None], (n_w, n, 1)))[:, :, 0]
    v = e + x @ K.T
    u = cbar[:, None] * a.conj()
    # LU with partial pivoting: relative error within a growth factor of the
    # order of n (random matrices: n^(2/3)) times n eps cond(A); forming
    # 1 - chi0 K adds n eps |chi0| |K|
    cond = np.linalg.cond(A).max()
    form = np.linalg.norm(chi0, 2, axis=(1, 2)).max() * np.linalg.norm(K, 2)
    inv = np.linalg.norm(np.linalg.inv(A), 2, axis=(1, 2)).max()
    tol = 4 * n * EPS * (n * cond + form * inv) + 64 * EPS
    dev = lambda z: torch.from_numpy(np.ascontiguousarray(z)).cuda()  # noqa: E731
    c, k, cb = dev(chi0), dev(K), dev(cbar)
    out = tdx.dyson(ctx, c, k, g0).cpu().numpy()
    assert np.max(np.abs(out - x[:, g0])) <= tol * np.max(np.linalg.norm(x, axis=1))
    gu, gv = (t.cpu().numpy() for t in tdx.dyson_vjp(ctx, c, k, g0, cb))
    assert np.max(np.linalg.norm(gu - u, axis=1)) <= tol * np.max(np.linalg.norm(u, axis=1))
    scale = np.linalg.norm(K, 2) * np.max(np.linalg.norm(x, axis=1)) + 1.0
    assert np.max(np.linalg.norm(gv - v, axis=1)) <= tol * scale


@pytest.mark.parametrize("n,col", [(5, 4), (16, 0), (16, 15), (40, 16), (40, 21), (130, 31),
                                   (130, 129), (260, 200), (305, 7)])
def test_vanishing_pivot_is_reported(tdx, ctx, n, col):
    """1 - chi0 K lower triangular with a zero on the diagonal: the elimination
    meets the zero column `col` exactly there."""
    import torch
    print("lu singular", n, col, flush=True)
    A = torch.eye(n, dtype=torch.complex128).repeat(3, 1, 1)
    A[1, col, col] = 0.0
    chi0 = (torch.eye(n, dtype=torch.complex128) - A).cuda().contiguous()
    K = torch.eye(n, dtype=torch.complex128).cuda()
    with pytest.raises(tdx.TdxError) as err:
        tdx.dyson(ctx, chi0, K, 0)
    assert err.value.code == tdx.ERR_NUMERIC
    assert f"frequency 1 (column {col})" in str(err.value)
    with pytest.raises(tdx.TdxError):
        tdx.dyson_vjp(ctx, chi0, K, 0, torch.ones(3, dtype=torch.complex128, device="cuda"))


@pytest.mark.parametrize("n", [33, 64, 133, 257, 304])
def test_back_substitution_keeps_small_products(tdx, ctx, n):
    """x_0 = (1 - sum_j u_0j x_j) / 2 with n - 1 products of 2^-54 each, every one
    of which a running difference from 1 would lose."""
    import torch
    print("lu small products", n, flush=True)
    chi0 = np.zeros((1, n, n), dtype=np.complex128)
    chi0[0, 1:, 0], chi0[0, 0, 1:], chi0[0, 0, 0] = 2.0 ** -20, 2.0 ** -33, 1.0
    K = -np.eye(n, dtype=np.complex128)
    A = (np.eye(n) + chi0[0]).real
    b = chi0[0, :, 0].real.astype(np.longdouble)
    x = np.linalg.solve(A, b.astype(np.float64)).astype(np.longdouble)
    for _ in range(3):
        x += np.linalg.solve(A, (b - A.astype(np.longdouble) @ x).astype(np.float64))
    got = tdx.dyson(ctx, torch.from_numpy(chi0).cuda(), torch.from_numpy(K).cuda(), 0)
    got = got.cpu().numpy()[0]
    # one rounding of half a unit for each block of 16 columns, six for the
    # elimination of the right-hand side and the quotient
    assert abs(np.longdouble(got.real) - x[0]) <= EPS * (n / 32 + 6) * x[0]
    assert got.imag == 0.0


@pytest.mark.parametrize("n,low,high", [(133, 5, 70), (257, 5, 256), (300, 40, 259), (304, 130, 300)])
def test_lowest_row_of_equal_pivots(tdx, ctx, n, low, high):
    """Rows `low` and `high` tie in the first column: x_0 + x_low = 0 and
    x_0 + 2^60 x_low = 2^60.  With the lower one first x_0 is -1 (to rounding);
    the other order subtracts 2^60 from itself and finds 0."""
    import torch
    print("lu tie", n, low, high, flush=True)
    A = np.eye(n)
    A[0, 0] = A[high, high] = 0.0
    A[low, 0] = A[high, 0] = A[0, high] = 1.0
    A[high, low] = 2.0 ** 60
    # 1 - chi0 K = A with K = -1; the right-hand side is column `low` of chi0 and
    # v = e_low + K x
    chi0 = torch.from_numpy((A - np.eye(n)).astype(np.complex128)[None]).cuda()
    K = torch.from_numpy(-np.eye(n, dtype=np.complex128)).cuda()
    cbar = torch.ones(1, dtype=torch.complex128, device="cuda")
    _, v = tdx.dyson_vjp(ctx, chi0, K, low, cbar)
    assert abs(complex(v[0, 0]) - 1.0) < 1e-12
