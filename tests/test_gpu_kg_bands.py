"""The Kubo-Greenwood conductivity by bands on seeded synthetic states: bands
around the groups of 5 and the tiles of 16, plane waves around the K-step of
16 and past what LDS holds, frequencies around the blocks of the sums, and
lists that are complete, hold one direction, miss transitions or are in
another order.  Reference: the defining sums, in FP64 on the CPU."""
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


def _system(tdx, npw, nb, seed):
    import torch
    rng = np.random.default_rng(seed)
    d = tdx.StatesDims()
    d.n_k, d.npw_max, d.nb_max = 2, npw + 3, nb
    st = tdx.States(d, 0)
    ax = np.arange(-6, 7)
    cube = np.stack(np.meshgrid(ax, ax, ax, indexing="ij"), -1).reshape(-1, 3)
    n = [npw, npw + 3]
    mil = np.zeros((2, npw + 3, 3), dtype=np.int32)
    coef = np.zeros((2, nb, npw + 3), dtype=np.complex128)
    for k in range(2):
        mil[k, :n[k]] = rng.permutation(cube)[:n[k]]
        coef[k, :, :n[k]] = rng.standard_normal((nb, n[k])) + 1j * rng.standard_normal((nb, n[k]))
    occ = np.where(np.arange(nb) < (nb + 1) // 2, rng.uniform(0.5, 1.0, (2, nb)), 0.0)
    eps = np.cumsum(rng.uniform(0.05, 0.2, (2, nb)), axis=1)
    for t, x in ((st.npw, np.array(n, dtype=np.int32)), (st.nb, np.full(2, nb, dtype=np.int32)),
                 (st.miller, mil), (st.eps, eps), (st.occ, occ), (st.coef, coef)):
        t.copy_(torch.from_numpy(x))
    b = rng.standard_normal((3, 3))
    st.c.kgrid[:] = [2, 1, 1]
    st.c.mmax[:] = [6, 6, 6]
    st.c.bvec[:] = list(b.reshape(-1))
    st.c.omega_cell = 37.0
    return st, n, mil, coef, b


def _list(tdx, tr, form, seed):
    """The list tr in another form: the kept transitions, in their order or not."""
    import torch
    T = len(tr)
    rng = np.random.default_rng(seed)
    keep = np.arange(T)
    n, m = tr.n.cpu().numpy(), tr.m.cpu().numpy()
    if form == "up":
        keep = keep[n[:T] < m[:T]]
    elif form == "down":
        keep = keep[n[:T] > m[:T]]
    elif form == "gaps":
        keep = keep[rng.random(T) < 0.6]
    elif form == "shuffled":
        keep = rng.permutation(T)
    out = tdx.Transitions(len(keep), 0)
    idx = torch.from_numpy(keep).cuda()
    for a in ("k", "n", "m", "delta", "df"):
        if len(keep):
            getattr(out, a).copy_(getattr(tr, a)[idx])
    return out


# (plane waves, bands, frequencies)
CASES = [(1, 2, 1), (15, 5, 7), (16, 6, 8), (17, 16, 9), (30, 17, 255), (33, 33, 257), (61, 40, 300),
         (1600, 7, 64)]


@pytest.mark.parametrize("form", ["full", "up", "down", "gaps", "shuffled"])
@pytest.mark.parametrize("npw,nb,n_w", CASES)
def test_conductivity_matches_the_defining_sums(tdx, ctx, npw, nb, n_w, form):
    import torch
    print("kg bands", npw, nb, n_w, form, flush=True)
    st, n, mil, coef, b = _system(tdx, npw, nb, 31 * npw + nb)
    tr = _list(tdx, tdx.transitions(ctx, st, (0, 0, 0), 1e-3), form, nb)
    T = len(tr)
    k, nn, mm = (x.cpu().numpy()[:T] for x in (tr.k, tr.n, tr.m))
    delta, df = tr.delta.cpu().numpy()[:T], tr.df.cpu().numpy()[:T]
    om, eta = np.linspace(-1.0, 3.0, n_w), 0.07
    W, mag = np.zeros(T), np.zeros(T)
    for t in range(T):
        kk = k[t]
        kf = mil[kk, :n[kk]] + np.array([(2.0 * kk - 1.0) / 4.0, 0.0, 0.0])
        g = kf @ b
        cm, cn = coef[kk, mm[t], :n[kk]], coef[kk, nn[t], :n[kk]]
        p = (np.conj(cm) * cn) @ g
        W[t] = df[t] / delta[t] * np.sum(np.abs(p) ** 2) / 3.0
        # the products' magnitudes, with those of the sums that make k + G
        a = np.abs(kf) @ np.abs(b)
        mag[t] = np.abs(df[t] / delta[t]) * np.sum((np.abs(cm) * np.abs(cn) @ a) ** 2) / 3.0
    pref = 2.0 / (37.0 * 2)
    den = om[:, None] - delta[None, :] + 1j * eta
    ref = 1j * pref * (W[None, :] / den).sum(axis=1)
    # |p|^2 as a sum of n terms on both sides (each relative error, then
    # squared), k + G and the weight's operations, the denominator's, the sum over t
    steps = 2 * (2 * (2 * (npw + 3) + 12)) + 40 + 2 * T
    tol = pref * steps * EPS * (mag[None, :] / np.abs(den)).sum(axis=1)
    got = tdx.kg_conductivity(ctx, st, torch.as_tensor(om, device="cuda"), eta, 1e-3,
                              tr=tr).cpu().numpy()
    assert np.all(np.abs(got - ref) <= tol), float(np.max(np.abs(got - ref) / (tol + 1e-300)))


def test_extreme_broadening_takes_the_division(tdx, ctx):
    """eta^2 under and over the range of the reciprocal estimate: all terms
    finite, sigma as the division gives it."""
    import torch
    st, *_ = _system(tdx, 17, 12, 5)
    tr = tdx.transitions(ctx, st, (0, 0, 0), 1e-3)
    om = torch.linspace(-1.0, 3.0, 33, device="cuda", dtype=torch.float64) + 1e-3
    base = tdx.kg_conductivity(ctx, st, om, 1e-9, 1e-3, tr=tr).cpu().numpy()
    tiny = tdx.kg_conductivity(ctx, st, om, 1e-150, 1e-3, tr=tr).cpu().numpy()
    # off the poles Im sigma depends on eta to O(eta^2 / x^2) only
    x = om.cpu().numpy()[:, None] - tr.delta.cpu().numpy()[None, :]
    assert np.min(np.abs(x)) > 1e-5
    scale = np.max(np.abs(base.imag))
    assert np.max(np.abs(tiny.imag - base.imag)) <= 1e-7 * scale
    huge = tdx.kg_conductivity(ctx, st, om, 1e145, 1e-3, tr=tr).cpu().numpy()
    assert np.all(np.isfinite(huge)) and np.max(np.abs(huge)) < 1e-140 * scale * 1e3


@pytest.mark.parametrize("npw", [31, 64, 250, 480])
def test_small_terms_of_a_momentum_element_are_kept(tdx, ctx, npw):
    """One plane wave holds 1 of p_mn, each other 2^-54: a sum in one go would
    lose them all."""
    import torch
    print("kg small terms", npw, flush=True)
    nb = 2
    d = tdx.StatesDims()
    d.n_k, d.npw_max, d.nb_max = 1, npw, nb
    st = tdx.States(d, 0)
    coef = np.zeros((1, nb, npw), dtype=np.complex128)
    coef[0, 1] = 1.0
    coef[0, 0] = 2.0 ** -54
    coef[0, 0, 0] = 1.0
    mil = np.zeros((1, npw, 3), dtype=np.int32)
    mil[..., 0] = 1
    for t, x in ((st.npw, np.array([npw], dtype=np.int32)), (st.nb, np.array([nb], dtype=np.int32)),
                 (st.miller, mil), (st.eps, np.array([[0.0, 0.5]])), (st.occ, np.array([[1.0, 0.0]])),
                 (st.coef, coef)):
        t.copy_(torch.from_numpy(x))
    st.c.kgrid[:] = [1, 1, 1]
    st.c.mmax[:] = [1, 1, 1]
    st.c.bvec[:] = [1.0, 0, 0, 0, 1.0, 0, 0, 0, 1.0]
    st.c.omega_cell = 1.0
    tr = tdx.transitions(ctx, st, (0, 0, 0), 1e-3)
    assert len(tr) == 2
    om = torch.linspace(0.0, 2.0, 40, dtype=torch.float64)
    eta = 0.25
    got = tdx.kg_conductivity(ctx, st, om.cuda(), eta, 1e-3, tr=tr).cpu().numpy()
    L = np.longdouble
    p2 = (1 + (npw - 1) * L(2) ** -54) ** 2
    x = om.numpy().astype(L)
    dl, df = tr.delta.cpu().numpy().astype(L), tr.df.cpu().numpy().astype(L)
    z = x[:, None] - dl + 1j * L(eta)
    ref = 2j * ((df / dl * p2 / 3) / z).sum(1)
    mag = 2 * (np.abs(df / dl * p2 / 3) / np.abs(z)).sum(1)
    # half a unit lost per term of the large one's own 32 and per later block,
    # twice as much of the square; 24 for the weight and its two quotients
    tol = EPS * (32 + npw / 32 + 24) * mag
    assert np.all(np.abs(got - ref) <= tol)


def _many_k(tdx, nk, nb, npw, seed, empty=()):
    """Seeded states on an nk x 1 x 1 grid; the k of `empty` have no transition."""
    import torch
    rng = np.random.default_rng(seed)
    d = tdx.StatesDims()
    d.n_k, d.npw_max, d.nb_max = nk, max(npw), nb
    st = tdx.States(d, 0)
    mil = rng.integers(-4, 5, (nk, max(npw), 3)).astype(np.int32)
    n = rng.choice(npw, nk).astype(np.int32)
    coef = rng.standard_normal((nk, nb, max(npw))) + 1j * rng.standard_normal((nk, nb, max(npw)))
    occ = np.where(np.arange(nb) < (nb + 1) // 2, rng.uniform(0.5, 1.0, (nk, nb)), 0.0)
    occ[list(empty)] = 0.0
    eps = np.cumsum(rng.uniform(0.05, 0.2, (nk, nb)), axis=1)
    for t, x in ((st.npw, n), (st.nb, np.full(nk, nb, dtype=np.int32)), (st.miller, mil),
                 (st.eps, eps), (st.occ, occ), (st.coef, coef)):
        t.copy_(torch.from_numpy(x))
    st.c.kgrid[:] = [nk, 1, 1]
    st.c.mmax[:] = [4, 4, 4]
    st.c.bvec[:] = [1.0, 0, 0, 0, 1.1, 0, 0, 0, 0.9]
    st.c.omega_cell = 37.0
    return st, n, mil, coef


@pytest.mark.parametrize("nk,nb", [(150, 23), (701, 7), (90, 41)])
def test_more_groups_of_bands_than_workgroups(tdx, ctx, nk, nb):
    """Two workgroups per CU take the groups of five bands in turn: more groups
    than those, eighths that are uneven, every seventh k without any."""
    import torch
    print("kg many k", nk, nb, flush=True)
    st, n, mil, coef = _many_k(tdx, nk, nb, (8, 13, 20), nk, range(0, nk, 7))
    tr = tdx.transitions(ctx, st, (0, 0, 0), 1e-3)
    T = len(tr)
    k, nn, mm = (x.cpu().numpy()[:T] for x in (tr.k, tr.n, tr.m))
    delta, df = tr.delta.cpu().numpy()[:T], tr.df.cpu().numpy()[:T]
    kf = mil + np.stack([(2.0 * np.arange(nk) + 1 - nk) / (2.0 * nk), 0 * np.arange(nk),
                         0 * np.arange(nk)], -1)[:, None]
    g = kf * np.array([1.0, 1.1, 0.9])
    live = np.arange(max(n)) < n[:, None]
    p = np.einsum("kmg,kga,kng->kanm", coef.conj() * live[:, None], g, coef)
    a = np.einsum("kmg,kga,kng->kanm", np.abs(coef) * live[:, None], np.abs(g), np.abs(coef))
    W = df / delta * (np.abs(p) ** 2).sum(1)[k, nn, mm] / 3.0
    mag = np.abs(df / delta) * (a ** 2).sum(1)[k, nn, mm] / 3.0
    om, eta = np.linspace(-1.0, 3.0, 160), 0.07
    # the list's table of rows and groups fits in the space of the partial sums,
    # and there are more groups than two workgroups on each of 256 CUs
    groups = nk * -(-nb // 5)
    assert 4 * (3 + nk * nb + groups) <= 16 * -(-T // 2048) * len(om) and groups * 6 // 7 > 512
    den = om[:, None] - delta[None, :] + 1j * eta
    pref = 2.0 / (37.0 * nk)
    ref = 1j * pref * (W[None, :] / den).sum(axis=1)
    steps = 2 * (2 * (2 * 20 + 12)) + 40 + 2 * T
    tol = pref * steps * EPS * (mag[None, :] / np.abs(den)).sum(axis=1)
    got = tdx.kg_conductivity(ctx, st, torch.as_tensor(om, device="cuda"), eta, 1e-3, tr=tr)
    assert np.all(np.abs(got.cpu().numpy() - ref) <= tol)


def test_a_shuffled_list_costs_its_weights_only(tdx, ctx):
    """The gaps between the rows of a list in another order are not filled: it
    takes about as long as one in which two transitions changed places."""
    import time

    import torch
    st, *_ = _many_k(tdx, 125, 160, (60,), 3)
    tr = tdx.transitions(ctx, st, (0, 0, 0), 1e-3)
    T = len(tr)
    print("kg shuffled", T, flush=True)
    om = torch.linspace(0.0, 2.0, 8, device="cuda", dtype=torch.float64)
    work = torch.empty(tdx.kg_work_bytes(T, 8), dtype=torch.uint8, device="cuda")
    us = []
    for perm in (np.r_[1, 0, 2:T], np.random.default_rng(1).permutation(T)):
        out = tdx.Transitions(T, 0)
        idx = torch.from_numpy(perm).cuda()
        for a in ("k", "n", "m", "delta", "df"):
            getattr(out, a).copy_(getattr(tr, a)[idx])
        best = 1e9
        for _ in range(5):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            tdx.kg_conductivity(ctx, st, om, 0.05, 1e-3, tr=out, work=work)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        us.append(1e6 * best)
    print(us, flush=True)
    assert us[1] < 4.0 * us[0]
