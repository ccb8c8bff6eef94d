"""Pair densities on seeded synthetic states at the edges of the shared-box
kernel: 1 to 10 tiles of 16 response vectors (one and two passes), groups of 1
to 40 transitions in row and column form, plane-wave counts around its K-step
of 4, response vectors whose reach is too wide for the padded lookup box, a
part of the list.  Reference: the defining sum, in FP64 on the CPU."""
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
    """States on a 2 x 1 x 1 grid: random bases, coefficients and occupations."""
    half = 4  # of the cube the plane waves come from: the smallest that holds them
    while (2 * half + 1) ** 3 < npw + 3:
        half += 1
    import torch
    rng = np.random.default_rng(seed)
    d = tdx.StatesDims()
    d.n_k, d.npw_max, d.nb_max = 2, npw + 3, nb
    st = tdx.States(d, 0)
    ax = np.arange(-half, half + 1)
    cube = np.stack(np.meshgrid(ax, ax, ax, indexing="ij"), -1).reshape(-1, 3)
    n = [npw, npw + 3]
    mil = np.zeros((2, npw + 3, 3), dtype=np.int32)
    coef = np.zeros((2, nb, npw + 3), dtype=np.complex128)
    for k in range(2):
        mil[k, :n[k]] = rng.permutation(cube)[:n[k]]
        coef[k, :, :n[k]] = rng.standard_normal((nb, n[k])) + 1j * rng.standard_normal((nb, n[k]))
    # a few bands occupied, the others below the screening: long rows of the
    # occupied bands, short rows (columns) of the empty ones
    occ = np.where(np.arange(nb) < 3, rng.uniform(0.5, 1.0, (2, nb)), 0.0)
    eps = np.sort(rng.standard_normal((2, nb)), axis=1)
    for t, x in ((st.npw, np.array(n, dtype=np.int32)), (st.nb, np.full(2, nb, dtype=np.int32)),
                 (st.miller, mil), (st.eps, eps), (st.occ, occ), (st.coef, coef)):
        t.copy_(torch.from_numpy(x))
    st.c.kgrid[:] = [2, 1, 1]
    st.c.mmax[:] = [half] * 3
    return st, n, mil, coef


# (plane waves, bands, response vectors, reach of the response vectors)
CASES = [(1, 4, 1, 1), (15, 40, 15, 2), (16, 17, 16, 3), (33, 18, 17, 2), (50, 40, 100, 3),
         (62, 24, 144, 4), (63, 20, 145, 4), (64, 33, 160, 5), (65, 30, 40, 120)]


@pytest.mark.parametrize("paired", [False, True])
@pytest.mark.parametrize("npw,nb,n_g,reach", CASES)
def test_pair_densities_match_the_defining_sum(tdx, ctx, npw, nb, n_g, reach, paired):
    import torch
    print("pair groups", npw, nb, n_g, reach, paired, flush=True)
    st, n, mil, coef = _system(tdx, npw, nb, 100 * npw + n_g)
    rng = np.random.default_rng(7 * n_g)
    near = rng.integers(-3, 4, (n_g, 3))
    far = rng.integers(-reach, reach + 1, (n_g, 3))
    basis = np.where(rng.random((n_g, 1)) < 0.5, near, far).astype(np.int32)
    qj = (1, 0, 2)
    tr = tdx.transitions(ctx, st, qj, 1e-3, paired=paired)
    T = len(tr)
    assert T > 0
    k, nn, mm = (x.cpu().numpy() for x in (tr.k, tr.n, tr.m))
    ref = np.zeros((T, n_g), dtype=np.complex128)
    mag = np.zeros((T, n_g))
    for kk in range(2):
        s = kk + qj[0]
        k2, gs = s % 2, np.array([s // 2, qj[1], qj[2]])
        where = {tuple(x): i for i, x in enumerate(mil[k2, :n[k2]])}
        sel = np.nonzero(k[:T] == kk)[0]
        for g in range(n_g):
            j = np.array([where.get(tuple(x + basis[g] + gs), -1) for x in mil[kk, :n[kk]]])
            b = np.where(j >= 0, coef[k2][:, np.maximum(j, 0)], 0.0)
            a = coef[kk][:, :n[kk]]
            ref[sel, g] = (a.conj() @ b.T)[nn[sel], mm[sel]]
            mag[sel, g] = (np.abs(a) @ np.abs(b).T)[nn[sel], mm[sel]]
    # four real products per plane wave, each rounded once when it is added
    tol = 4 * EPS * (npw + 8) * 2 * mag
    gb = torch.from_numpy(basis).cuda()
    P = tdx.pair_density(ctx, st, qj, tr, gb, "fp64")
    got = tdx.pair_density_view(P, T, n_g, "fp64").cpu().numpy()
    assert np.all(np.abs(got - ref) <= tol)
    ld = (n_g + 15) // 16 * 16
    whole = P[: T * ld * 16].view(torch.complex128).view(T, ld)
    assert not torch.any(whole[:, n_g:])
    # a part of the list cuts groups elsewhere, so a transition may be summed
    # over the other side's plane waves: the same bound
    b0, b1 = T // 3, max(T // 3 + 1, 2 * T // 3)
    part = tdx.pair_density_range(ctx, st, qj, tr, gb, b0, b1, "fp64")
    part = tdx.pair_density_view(part, b1 - b0, n_g, "fp64").cpu().numpy()
    assert np.all(np.abs(part - ref[b0:b1]) <= tol[b0:b1])
    p32 = tdx.pair_density_view(tdx.pair_density(ctx, st, qj, tr, gb, "fp32"), T, n_g, "fp32")
    assert torch.equal(p32, whole[:, :n_g].to(torch.complex64))


# one group per workgroup, which runs where the shared form's fixed sides and box
# do not fit: plane waves on either side of that line, then one wavefront with
# the Miller indices in LDS, eight with them, eight without; and either side of
# 96 plane waves at one tile of response vectors
@pytest.mark.parametrize("paired", [False, True])
@pytest.mark.parametrize("npw,nb,n_g,reach",
                         [(1214, 5, 17, 3), (1215, 5, 17, 3), (1400, 7, 33, 4), (3000, 6, 17, 3),
                          (6350, 5, 16, 3), (93, 30, 16, 3), (94, 30, 16, 3)])
def test_larger_bases_match_the_defining_sum(tdx, ctx, npw, nb, n_g, reach, paired):
    test_pair_densities_match_the_defining_sum(tdx, ctx, npw, nb, n_g, reach, paired)
