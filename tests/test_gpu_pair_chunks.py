"""Pair densities of lists with more chunks than workgroups, which take the
next chunk of any k-point from a counter: three k-points, one without
transitions; chunks of one tile and of eight; rows and, for a few occupied
bands, columns.  Reference: the defining sum, in FP64 on the CPU."""
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


# (plane waves, bands, occupied bands with a spread of occupations, response vectors)
CASES = [(12, 70, 70, 5), (9, 900, 24, 17), (20, 180, 180, 2)]


@pytest.mark.parametrize("npw,nb,occupied,n_g", CASES)
def test_pair_densities_match_the_defining_sum(tdx, npw, nb, occupied, n_g):
    import torch
    print("pair chunks", npw, nb, occupied, n_g, flush=True)
    rng = np.random.default_rng(npw)
    d = tdx.StatesDims()
    d.n_k, d.npw_max, d.nb_max = 3, npw, nb
    st = tdx.States(d, 0)
    cube = np.stack(np.meshgrid(*[np.arange(-2, 3)] * 3, indexing="ij"), -1).reshape(-1, 3)
    mil = np.stack([rng.permutation(cube)[:npw] for _ in range(3)]).astype(np.int32)
    coef = rng.standard_normal((3, nb, npw)) + 1j * rng.standard_normal((3, nb, npw))
    occ = np.zeros((3, nb))
    occ[:, :occupied] = rng.uniform(0.5, 1.0, (3, occupied))
    # q takes k = 1 to k = 2: none of their differences passes
    occ[1:] = 0.25
    eps = np.sort(rng.standard_normal((3, nb)), axis=1)
    for t, x in ((st.npw, np.full(3, npw, dtype=np.int32)), (st.nb, np.full(3, nb, dtype=np.int32)),
                 (st.miller, mil), (st.eps, eps), (st.occ, occ), (st.coef, coef)):
        t.copy_(torch.from_numpy(x))
    st.c.kgrid[:] = [3, 1, 1]
    st.c.mmax[:] = [2, 2, 2]
    qj = (1, 0, 0)
    basis = rng.integers(-2, 3, (n_g, 3)).astype(np.int32)
    ctx = tdx.Context(0)
    tr = tdx.transitions(ctx, st, qj, 1e-3)
    T = len(tr)
    k, nn, mm = (x.cpu().numpy()[:T] for x in (tr.k, tr.n, tr.m))
    assert T / 16 > 256 and not np.any(k == 1) and np.any(k == 0) and np.any(k == 2)
    got = tdx.pair_density_view(tdx.pair_density(ctx, st, qj, tr, torch.from_numpy(basis).cuda(),
                                                 "fp64"), T, n_g, "fp64").cpu().numpy()
    for kk in (0, 2):
        k2, gs = (kk + 1) % 3, np.array([(kk + 1) // 3, 0, 0])
        where = {tuple(x): i for i, x in enumerate(mil[k2])}
        sel = np.nonzero(k == kk)[0]
        for g in range(n_g):
            j = np.array([where.get(tuple(x + basis[g] + gs), -1) for x in mil[kk]])
            b = np.where(j >= 0, coef[k2][:, np.maximum(j, 0)], 0.0)
            a = coef[kk]
            ref = (a.conj() @ b.T)[nn[sel], mm[sel]]
            mag = (np.abs(a) @ np.abs(b).T)[nn[sel], mm[sel]]
            # four real products per plane wave, each rounded once when added
            assert np.all(np.abs(got[sel, g] - ref) <= 4 * EPS * (npw + 8) * 2 * mag)
    ctx.close()


# plane waves times tiles of 16 response vectors just above 96 and above 600
@pytest.mark.parametrize("npw,nb,occupied,n_g",
                         [(100, 70, 70, 97), (49, 900, 24, 17), (97, 180, 180, 2)])
def test_larger_bases_match_the_defining_sum(tdx, npw, nb, occupied, n_g):
    test_pair_densities_match_the_defining_sum(tdx, npw, nb, occupied, n_g)


@pytest.mark.parametrize("n_g", [15, 129])
def test_a_list_of_short_rows_takes_no_longer_than_one_of_long_rows(tdx, n_g):
    """512 k of 52 plane waves and 12 bands: eleven tiles of one transition each
    against twelve of eleven."""
    import time

    import torch
    nk, npw, nb = 512, 52, 12
    rng = np.random.default_rng(n_g)
    cube = np.stack(np.meshgrid(*[np.arange(-2, 3)] * 3, indexing="ij"), -1).reshape(-1, 3)
    cube = cube[np.argsort((cube ** 2).sum(1), kind="stable")]
    ctx = tdx.Context(0)
    us = []
    for occupied in (1, nb):
        d = tdx.StatesDims()
        d.n_k, d.npw_max, d.nb_max = nk, npw, nb
        st = tdx.States(d, 0)
        coef = rng.standard_normal((nk, nb, npw)) + 1j * rng.standard_normal((nk, nb, npw))
        occ = np.zeros((nk, nb))
        occ[:, :occupied] = rng.uniform(0.5, 1.0, (nk, occupied))
        eps = np.sort(rng.standard_normal((nk, nb)), axis=1)
        for t, x in ((st.npw, np.full(nk, npw, dtype=np.int32)),
                     (st.nb, np.full(nk, nb, dtype=np.int32)),
                     (st.miller, np.stack([cube[:npw]] * nk).astype(np.int32)),
                     (st.eps, eps), (st.occ, occ), (st.coef, coef)):
            t.copy_(torch.from_numpy(x))
        st.c.kgrid[:] = [8, 8, 8]
        st.c.mmax[:] = [2, 2, 2]
        basis = torch.from_numpy(rng.integers(-2, 3, (n_g, 3)).astype(np.int32)).cuda()
        tr = tdx.transitions(ctx, st, (0, 1, 1), 1e-3, paired=False)
        out = torch.empty(tdx.pair_density_bytes(len(tr), n_g, "fp64"), dtype=torch.uint8,
                          device="cuda")
        best = 1e9
        for _ in range(8):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(5):
                tdx.pair_density(ctx, st, (0, 1, 1), tr, basis, "fp64", out=out)
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - t0) / 5)
        us.append(1e6 * best)
        print("short rows", n_g, occupied, len(tr), us, flush=True)
    ctx.close()
    assert us[0] < 1.2 * us[1]
