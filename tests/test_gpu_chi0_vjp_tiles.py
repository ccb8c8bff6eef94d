"""The cotangents of chi0 at the edges of their tiles: response vectors around
each register layout (and past the largest), transitions around the tile of 16
and past what one round of workgroups takes, frequencies around the tile of 16,
full and paired lists, with and without the pair-density cotangent, a part of
a list.  Reference: the defining sums, in FP64 on the CPU."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -53
ETA, PREF = 0.06, 0.013


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


# (response vectors, transitions, frequencies)
CASES = [(1, 1, 1), (15, 16, 15), (16, 17, 16), (17, 31, 17), (48, 33, 129), (49, 130, 33),
         (96, 40, 31), (97, 15, 64), (144, 17, 130), (145, 50, 40), (192, 65, 7), (193, 16, 33),
         (256, 20, 65), (257, 33, 16), (320, 18, 17), (321, 40, 18), (20, 9000, 24)]


@pytest.mark.parametrize("paired", [False, True])
@pytest.mark.parametrize("n_g,n_t,n_w", CASES)
def test_cotangents_match_the_defining_sums(tdx, ctx, n_g, n_t, n_w, paired):
    import torch
    print("chi0 vjp tiles", n_g, n_t, n_w, paired, flush=True)
    rng = np.random.default_rng(1000 * n_g + n_t)
    cn = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)  # noqa: E731
    skip = 3  # transitions of the list before the part that is asked for
    tr = tdx.Transitions(n_t + skip, 0, paired=paired)
    dl, df = rng.uniform(0.05, 1.5, n_t + skip), rng.uniform(0.1, 1.0, n_t + skip)
    tr.delta.copy_(torch.from_numpy(dl))
    tr.df.copy_(torch.from_numpy(df))
    dl, df = dl[skip:], df[skip:]
    ld = (n_g + 15) // 16 * 16
    P = np.zeros((n_t, ld), dtype=np.complex128)
    P[:, :n_g] = rho = cn(n_t, n_g)
    u, v, om = cn(n_w, n_g), cn(n_w, n_g), np.linspace(0.0, 2.0, n_w)
    a, b = np.conj(u) @ rho.T, np.conj(v) @ rho.T  # [n_w, n_t]
    r1 = 1.0 / (om[:, None] - dl[None, :] + 1j * ETA)
    r2 = 1.0 / (om[:, None] + dl[None, :] + 1j * ETA) if paired else np.zeros_like(r1)
    lam = PREF * a * np.conj(b)
    w_ref = np.stack([(lam * (r1 - r2)).sum(0).real, df * (lam * (r1 ** 2 + r2 ** 2)).sum(0).real,
                      df * (-1j * lam * (r1 ** 2 - r2 ** 2)).sum(0).real], axis=1)
    w = df[None, :] * (r1 - r2)
    c1, c2 = PREF * w * np.conj(b), PREF * w * a
    rho_ref = np.conj(c1).T @ u + c2.T @ v
    # magnitudes of the terms; per term two sums of n_g complex products and
    # the weight's operations, then the sum over frequencies, on both sides
    A, B = np.abs(u) @ np.abs(rho).T, np.abs(v) @ np.abs(rho).T
    R1, R2 = np.abs(r1) + np.abs(r2), np.abs(r1) ** 2 + np.abs(r2) ** 2
    L = PREF * A * B
    steps = 2 * (2 * (2 * n_g + 8) + 40 + n_w)
    w_tol = steps * EPS * np.stack([(L * R1).sum(0), df * (L * R2).sum(0), df * (L * R2).sum(0)], 1)
    steps = 2 * ((2 * n_g + 8) + 40 + 4 * n_w)
    C = PREF * df[None, :] * R1
    rho_tol = steps * EPS * ((C * B).T @ np.abs(u) + (C * A).T @ np.abs(v))
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    Pd, ud, vd, od = dev(P), dev(u), dev(v), dev(om)
    for want in (True, False):
        w_bar, rho_bar = tdx.chi0_vjp(ctx, tr, Pd, n_g, od, ETA, PREF, ud, vd, want_rho=want,
                                      t_begin=skip)
        assert np.all(np.abs(w_bar.cpu().numpy() - w_ref) <= w_tol)
        if want:
            got = rho_bar.cpu().numpy()
            assert got.shape == (n_t, ld)
            assert np.all(np.abs(got[:, :n_g] - rho_ref) <= rho_tol)
            assert np.all(got[:, n_g:] == 0.0)
        else:
            assert rho_bar is None


def test_more_transitions_than_one_tile_each_launches(tdx, ctx):
    """2^27 + 5 transitions, all alike: with 16 of them per workgroup of 512
    threads the launch would hold 2^32 threads."""
    import torch
    n_t, n_g, n_w = (1 << 27) + 5, 2, 128
    print("vjp many transitions", n_t, flush=True)
    if torch.cuda.mem_get_info()[0] < (48 << 30):
        pytest.skip("needs 48 GiB")
    rng = np.random.default_rng(1)
    u, v = (rng.standard_normal((n_w, n_g)) + 1j * rng.standard_normal((n_w, n_g)) for _ in range(2))
    om = np.linspace(0.0, 2.0, n_w)
    dl, df, rho = 0.7, 0.4, np.array([1.0 + 0.5j, -0.25 + 2.0j])
    tr = tdx.Transitions(n_t, 0, paired=False)
    tr.delta.fill_(dl)
    tr.df.fill_(df)
    P = torch.zeros(n_t, 16, dtype=torch.complex128, device="cuda")
    P[:, 0], P[:, 1] = complex(rho[0]), complex(rho[1])
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    w_bar, _ = tdx.chi0_vjp(ctx, tr, P, n_g, dev(om), ETA, PREF, dev(u), dev(v))
    del P
    al, be = u.conj() @ rho, v.conj() @ rho
    r = 1.0 / (om - dl + 1j * ETA)
    lam = PREF * al * be.conj()
    want = np.array([(lam * r).real.sum(), df * (lam * r * r).real.sum(), df * (lam * r * r).imag.sum()])
    # products of sums of n_g terms, their weights and the sum over frequencies
    mag = np.abs(PREF) * (np.abs(u) @ np.abs(rho)) * (np.abs(v) @ np.abs(rho)) * np.abs(r)
    tol = 2 * EPS * (n_w + 40) * np.array([mag.sum(), df * (mag * np.abs(r)).sum(),
                                           df * (mag * np.abs(r)).sum()])
    bad = (w_bar - dev(want)).abs() > dev(tol)
    assert not bool(bad.any())


@pytest.mark.parametrize("n_g", [20, 60, 133, 190, 250, 300])
def test_no_sum_of_rhobar_is_longer_than_64_frequencies(tdx, ctx, n_g):
    """The first frequency gives 1 of rhobar, each other 2^-54 of it: those of the
    first one's sum are lost, the others' sums kept."""
    import torch
    n_t, n_w = 40, 4000
    print("vjp sum length", n_g, flush=True)
    tr = tdx.Transitions(n_t, 0, paired=False)
    tr.delta.fill_(0.7)
    tr.df.fill_(0.5)
    ld = (n_g + 15) // 16 * 16
    P = torch.zeros(n_t, ld, dtype=torch.complex128, device="cuda")
    P[:, 0] = 1.0
    u = torch.zeros(n_w, n_g, dtype=torch.complex128, device="cuda")
    v = torch.zeros_like(u)
    u[:, 0], u[0, 0], v[:, 0] = 2.0 ** -54, 1.0, 1.0
    om = torch.full((n_w,), 0.25, dtype=torch.float64, device="cuda")
    _, rho_bar = tdx.chi0_vjp(ctx, tr, P, n_g, om, ETA, PREF, u, v, want_rho=True)
    # alpha = u, beta = v = 1: rhobar_0 = sum_w 2 pref Re(w_t) u
    x = np.longdouble(0.25) - np.longdouble(0.7)
    r = np.longdouble(0.5) * x / (x * x + np.longdouble(ETA) ** 2)
    ref = 2 * np.longdouble(PREF) * r * (1 + (n_w - 1) * np.longdouble(2) ** -54)
    got = rho_bar.cpu().numpy()[:, 0].real
    # half a unit for each of the 63, one per later sum of 64 and per wave, 16 for
    # the weight and its products
    tol = EPS * (32 + n_w / 64 + 8 + 16) * abs(ref)
    assert np.all(np.abs(got - ref) <= tol)
