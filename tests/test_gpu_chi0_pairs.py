"""The FP64 chi0 contraction over pairs G <= G' at the edges of its tiles:
16 frequencies a block, 64 or 128 pairs a tile, 16 transitions a chunk, one
slice and several, both list forms, every tile variant.  Reference: the sum
over transitions in plain torch, FP64, on the CPU."""
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


# (n_g, n_w, n_trans, fixed slice length or 0)
CASES = [(1, 1, 1, 0), (2, 15, 15, 0), (10, 16, 16, 0), (11, 17, 17, 16), (15, 33, 31, 16),
         (16, 48, 32, 0), (17, 49, 95, 48), (33, 64, 65, 32), (45, 80, 200, 0), (23, 129, 47, 0)]


@pytest.mark.parametrize("paired", [True, False])
@pytest.mark.parametrize("n_g,n_w,n_t,slice_len", CASES)
def test_pair_tiles_match_the_plain_sum(tdx, ctx, n_g, n_w, n_t, slice_len, paired):
    import torch
    print("pairs", n_g, n_w, n_t, slice_len, paired, flush=True)
    g = torch.Generator().manual_seed(1000 * n_g + n_t)
    rho = torch.randn(n_t, n_g, generator=g, dtype=torch.complex128)
    delta = torch.randn(n_t, generator=g, dtype=torch.float64)
    df = torch.randn(n_t, generator=g, dtype=torch.float64)
    om = torch.linspace(0.0, 2.0, n_w, dtype=torch.float64)
    eta, pref = 0.05, 0.7
    z = (om + 1j * eta)[:, None]
    w = 2 * df * delta / ((om[:, None] - delta) * (om[:, None] + delta) - eta * eta
                          + 2j * om[:, None] * eta) if paired else df / (z - delta)
    X = (rho[:, :, None] * rho.conj()[:, None, :]).reshape(n_t, -1)
    ref = (pref * (w @ X)).view(n_w, n_g, n_g)
    # a sum of n_t products, each of a rounded weight (about 12 roundings) and a
    # rounded product of rho (3): n_t + 16 roundings of the sum of magnitudes in
    # either order of the sum; twice that for the difference of two such sums,
    # and twice again for the real and imaginary parts held apart
    mag = (abs(pref) * (w.abs() @ X.abs())).view(n_w, n_g, n_g)
    tol = 4 * EPS * (n_t + 16) * mag

    tr = tdx.Transitions(n_t, 0, paired)
    tr.delta.copy_(delta)
    tr.df.copy_(df)
    ld = (n_g + 15) // 16 * 16
    P = torch.zeros(n_t, ld, dtype=torch.complex128)
    P[:, :n_g] = rho
    P = torch.view_as_real(P.cuda()).reshape(-1).view(torch.uint8)
    tdx.chi0_set_slice_length(ctx, slice_len)
    try:
        for v in [-1] + list(range(tdx.chi0_variants("fp64"))):
            tdx.chi0_set_config(ctx, n_g, v, 20, "fp64")
            out = torch.full((n_w, n_g, n_g), complex("nan"), dtype=torch.complex128, device="cuda")
            tdx.chi0(ctx, tr, P, n_g, "fp64", om.cuda(), eta, pref, out=out)
            err = (out.cpu() - ref).abs()
            assert bool((err <= tol).all()), (v, float((err / mag).max()))
    finally:
        tdx.chi0_set_slice_length(ctx, 0)
        tdx.chi0_set_config(ctx, n_g, -1, 20, "fp64")


def _uniform(tdx, n_g, n_t, df):
    """A list whose transitions all sit at delta = 0.3, with rho = 1 everywhere."""
    import torch
    tr = tdx.Transitions(n_t, 0, False)
    tr.delta.fill_(0.3)
    tr.df.copy_(df)
    P = torch.zeros(n_t, (n_g + 15) // 16 * 16, dtype=torch.complex128, device="cuda")
    P[:, :n_g] = 1.0
    return tr, torch.view_as_real(P).reshape(-1).view(torch.uint8)


@pytest.mark.parametrize("n_g,n_w,n_t", [(94, 40, 44838), (75, 60, 20000), (20, 40, 9000), (144, 40, 1000)])
def test_no_sum_is_longer_than_two_of_the_slices(tdx, ctx, n_g, n_w, n_t):
    """One large term first and then terms of 2^-54 of it, each of which a sum
    that holds the large one loses: the loss bounds the length of that sum."""
    import numpy as np
    import torch
    print("sum length", n_g, n_w, n_t, flush=True)
    df = torch.full((n_t,), 2.0 ** -54, dtype=torch.float64)
    df[0] = 1.0
    tr, P = _uniform(tdx, n_g, n_t, df)
    om = torch.linspace(0.0, 2.0, n_w, dtype=torch.float64)
    eta = 0.05
    out = tdx.chi0(ctx, tr, P, n_g, "fp64", om.cuda(), eta, 1.0).cpu().numpy()
    x = om.numpy().astype(np.longdouble) - np.longdouble(0.3)
    ref = x / (x * x + np.longdouble(eta) ** 2) * (1 + np.longdouble(n_t - 1) * np.longdouble(2) ** -54)
    ld = (n_g + 15) // 16 * 16
    slices = min(-(-4096 // (-(-n_w // 8) * (ld // 16) * -(-ld // 48))), -(-n_t // 16))
    # the terms lost by a sum of twice those of equal slices (half a unit
    # each), the sum over slices, and the roundings of the weight (12)
    tol = EPS * (n_t / slices + 32 + slices + 12)
    got = out.real.astype(np.longdouble)
    assert np.all(np.abs(got - ref[:, None, None]) <= tol * np.abs(ref)[:, None, None])


def test_a_limit_set_after_use_leaves_room(tdx):
    """The partials of a contraction without a limit are no larger than those of
    one with it: what fitted beside them still does."""
    import torch
    n_g, n_w, n_t = 133, 500, 50000
    print("limit after use", n_g, n_w, n_t, flush=True)
    c = tdx.Context(0)
    tr, P = _uniform(tdx, n_g, n_t, torch.full((n_t,), 1.0 / n_t, dtype=torch.float64))
    om = torch.linspace(0.0, 2.0, n_w, dtype=torch.float64).cuda()
    chi0 = tdx.chi0(c, tr, P, n_g, "fp64", om, 0.05, 1.0)
    torch.cuda.synchronize()
    mat = 16 * n_w * n_g * n_g
    c.set_workspace_limit(4 * mat + 4096)  # three slices and the Dyson matrices
    K = torch.eye(n_g, dtype=torch.complex128, device="cuda") * 1e-3
    tdx.dyson(c, chi0, K, 0)
    c.close()


def test_more_tiles_than_one_axis_of_a_launch_holds(tdx, ctx):
    """65535 slices of 157 frequency tiles each, 5.3e9 threads."""
    import numpy as np
    import torch
    n_w, n_t, eta = 10000, 16 * 65535, 0.05
    print("many tiles", n_w, n_t, flush=True)
    tr, P = _uniform(tdx, 1, n_t, torch.full((n_t,), 1.0, dtype=torch.float64))
    om = torch.linspace(0.0, 2.0, n_w, dtype=torch.float64)
    c = tdx.Context(0)
    tdx.chi0_set_slice_length(c, 16)
    tdx.chi0_set_config(c, 1, 0, 20, "fp64")
    out = tdx.chi0(c, tr, P, 1, "fp64", om.cuda(), eta, 1.0).cpu().numpy().reshape(-1)
    c.close()
    ref = n_t / (om.numpy() - 0.3 + 1j * eta)
    assert np.all(np.abs(out - ref) <= 2 * EPS * (16 + 65535 + 16) * np.abs(ref))
