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
