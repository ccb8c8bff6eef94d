"""Several spectra through the Laplace transform in one launch: each row equal
to the single call bit for bit, at set counts around the eight of a block and
frequency counts around its 1024-value chunk; the single call against the
defining sum."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_set,n_w,n_tau", [(0, 5, 3), (1, 2, 1), (2, 63, 2), (7, 500, 65),
                                             (8, 1024, 3), (9, 1025, 5), (17, 2100, 4)])
def test_rows_equal_single_calls(n_set, n_w, n_tau):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_01875_amd as tdx
    print("itcf sets", n_set, n_w, n_tau, flush=True)
    ctx = tdx.Context(0)
    rng = np.random.default_rng(n_w)
    om = np.cumsum(rng.uniform(0.5, 1.5, n_w)) * (2.0 / n_w)
    beta = 20.0
    tau = np.linspace(0.0, beta, n_tau)
    S = rng.standard_normal((n_set, n_w))
    dev = lambda x: torch.from_numpy(x).cuda()  # noqa: E731
    F = tdx.itcf_sets(ctx, dev(S), dev(om), beta, dev(tau))
    assert F.shape == (n_set, n_tau)
    c = np.zeros(n_w)
    c[1:] += 0.5 * np.diff(om)
    c[:-1] += 0.5 * np.diff(om)
    e = c * (np.exp(-np.outer(tau, om)) + np.exp(-np.outer(beta - tau, om)))
    # n_w products summed, each exponential within 2 ulp of an argument rounded
    # once (at most beta * max(om) in size)
    tol = 2.0 ** -53 * (n_w + 8 + 2 * beta * om[-1]) * (np.abs(S) @ np.abs(e).T)
    assert np.all(np.abs(F.cpu().numpy() - S @ e.T) <= tol)
    for i in range(n_set):
        assert torch.equal(F[i], tdx.itcf(ctx, dev(S[i].copy()), dev(om), beta, dev(tau)))
    ctx.close()


@pytest.mark.parametrize("n_set,n_w", [(1, 100001), (2, 100001), (6, 20000), (1, 8193), (9, 4097)])
def test_strides_of_long_grids(n_set, n_w):
    """Sixty-four large terms and then small ones of 2^-54 of them: 256 strides
    lose a quarter of these (in one wave's 64, all of them)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_01875_amd as tdx
    print("itcf strides", n_set, n_w, flush=True)
    ctx = tdx.Context(0)
    om = torch.arange(n_w, dtype=torch.float64) * 2.0 ** -10
    tau = torch.zeros(1, dtype=torch.float64)
    S = torch.full((n_set, n_w), 2.0 ** -54, dtype=torch.float64)
    S[:, :64] = 1.0
    # beta so small that each exponential is 1: the weight is twice the step,
    # half of that at the ends
    F = tdx.itcf_sets(ctx, S.cuda(), om.cuda(), 1e-30, tau.cuda()).cpu().numpy()[:, 0]
    ctx.close()
    ref = (np.longdouble(63.5) + (n_w - 64 - np.longdouble(0.5)) * np.longdouble(2) ** -54) * 2.0 ** -9
    # 2^-54 lost for a third of the terms at most; eight roundings of the tree
    tol = (n_w / 3 * 2.0 ** -54 + 8 * 2.0 ** -53 * 64) * 2.0 ** -9
    assert np.all(np.abs(F - ref) <= tol)
