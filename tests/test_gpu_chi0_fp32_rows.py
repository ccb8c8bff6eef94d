"""FP32 chi0 at the edges of the tiles that hold all columns: bases around each
count of 16-column blocks and past the last, rows (frequency, vector) that end
inside and at a tile, lists around the chunk of 32 transitions, past a run of
4096 and in several slices, full and paired.  Reference: the defining sum in
FP64 on the CPU."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24
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


# (vectors, frequencies, transitions)
CASES = [(16, 9, 40), (17, 1, 1), (31, 13, 33), (32, 12, 32), (33, 40, 31), (48, 11, 100),
         (49, 3, 65), (64, 16, 64), (65, 7, 4097), (80, 5, 96), (81, 4, 50), (96, 6, 33),
         (97, 9, 8200), (112, 8, 40), (113, 5, 70), (128, 2, 129), (129, 3, 31), (144, 4, 64),
         (145, 3, 40)]


@pytest.mark.parametrize("paired", [False, True])
@pytest.mark.parametrize("n_g,n_w,n_t", CASES)
def test_chi0_matches_the_defining_sum(tdx, ctx, n_g, n_w, n_t, paired):
    import torch
    print("chi0 fp32 rows", n_g, n_w, n_t, paired, flush=True)
    rng = np.random.default_rng(100 * n_g + n_t)
    tr = tdx.Transitions(n_t, 0, paired=paired)
    dl, df = rng.uniform(0.05, 1.5, n_t), rng.uniform(0.1, 1.0, n_t)
    tr.delta.copy_(torch.from_numpy(dl))
    tr.df.copy_(torch.from_numpy(df))
    ld = (n_g + 15) // 16 * 16
    P = np.zeros((n_t, ld), dtype=np.complex64)
    P[:, :n_g] = rng.standard_normal((n_t, n_g)) + 1j * rng.standard_normal((n_t, n_g))
    rho = P[:, :n_g].astype(np.complex128)
    om = np.linspace(0.0, 2.0, n_w)
    w = df / (om[:, None] - dl + 1j * ETA)
    if paired:
        w = w - df / (om[:, None] + dl + 1j * ETA)
    ref = np.stack([PREF * (rho.T * wi) @ rho.conj() for wi in w])
    a = np.abs(rho)
    # FP32: the weight (8 operations), w rho, and a run of at most 4096
    # transitions (two products each for Re and Im)
    steps = 2 * (2 * min(n_t, 4096) + 12)
    tol = steps * EPS * np.stack([PREF * (a.T * wi) @ a for wi in np.abs(w)])
    Pd = torch.from_numpy(P).cuda()
    got = tdx.chi0(ctx, tr, Pd, n_g, "fp32", torch.from_numpy(om).cuda(), ETA, PREF)
    assert np.all(np.abs(got.cpu().numpy().reshape(ref.shape) - ref) <= tol)


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("n_g,n_t", [(48, 33), (64, 5), (113, 40), (144, 70)])
def test_a_value_that_is_not_finite_stays_in_its_row_and_column(tdx, ctx, n_g, n_t, bad):
    """The last transition's last vector, in a list that ends inside a chunk:
    every entry outside that vector's row and column is the one of a list with
    a zero in its place."""
    import torch
    print("chi0 fp32 rows, not finite", n_g, n_t, bad, flush=True)
    n_w = 5
    rng = np.random.default_rng(n_g + n_t)
    tr = tdx.Transitions(n_t, 0, paired=True)
    tr.delta.copy_(torch.from_numpy(rng.uniform(0.05, 1.5, n_t)))
    tr.df.copy_(torch.from_numpy(rng.uniform(0.1, 1.0, n_t)))
    P = np.zeros((n_t, (n_g + 15) // 16 * 16), dtype=np.complex64)
    P[:, :n_g] = rng.standard_normal((n_t, n_g)) + 1j * rng.standard_normal((n_t, n_g))
    om = torch.linspace(0.0, 2.0, n_w, dtype=torch.float64).cuda()
    out = []
    for x in (0.0, bad):
        P[-1, n_g - 1] = x
        out.append(tdx.chi0(ctx, tr, torch.from_numpy(P).cuda(), n_g, "fp32", om, ETA, PREF)
                   .cpu().numpy().reshape(n_w, n_g, n_g))
    assert np.array_equal(out[0][:, :-1, :-1], out[1][:, :-1, :-1])
    assert not np.isfinite(out[1][:, -1, -1]).any()


# lists on which the all-column tiles run, and, in several chunks, slices and
# tiles, those on which the general tiles do
@pytest.mark.parametrize("paired", [False, True])
@pytest.mark.parametrize("n_g,n_w,n_t",
                         [(17, 1, 5001), (29, 60, 5000), (31, 60, 5000), (33, 5, 5003),
                          (48, 11, 8200), (80, 5, 1040), (113, 5, 731), (128, 2, 705),
                          (129, 3, 331), (144, 4, 8200), (16, 40, 300), (29, 60, 1666),
                          (29, 60, 1667), (30, 60, 8200), (32, 40, 300), (48, 40, 999),
                          (48, 40, 1000), (80, 13, 999), (80, 13, 1000), (128, 10, 399),
                          (128, 10, 400), (144, 4, 299), (144, 4, 300), (145, 20, 100)])
def test_chi0_of_other_lists_matches_the_defining_sum(tdx, ctx, n_g, n_w, n_t, paired):
    test_chi0_matches_the_defining_sum(tdx, ctx, n_g, n_w, n_t, paired)


# several chunks, columns that end inside a tile of each variant
@pytest.mark.parametrize("variant", range(5))
@pytest.mark.parametrize("n_g,n_w,n_t", [(16, 33, 300), (32, 20, 200), (48, 17, 130),
                                         (80, 5, 99), (145, 9, 100), (180, 3, 65)])
def test_every_variant_of_the_general_tiles_matches_the_defining_sum(tdx, n_g, n_w, n_t, variant):
    assert tdx.chi0_variants("fp32") == 5
    c = tdx.Context(0)
    tdx.chi0_set_config(c, n_g, variant, 20, "fp32")
    assert tdx.chi0_get_config(c, n_g, "fp32")[0] == variant
    test_chi0_matches_the_defining_sum(tdx, c, n_g, n_w, n_t, True)
    c.close()


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("n_g,n_t", [(20, 5003), (48, 8005), (80, 1001), (128, 805), (144, 333)])
def test_a_value_that_is_not_finite_stays_in_place_in_longer_lists(tdx, ctx, n_g, n_t, bad):
    test_a_value_that_is_not_finite_stays_in_its_row_and_column(tdx, ctx, n_g, n_t, bad)


@pytest.mark.parametrize("n_w", [20, 80])
def test_a_short_list_of_29_vectors_takes_no_longer_than_one_of_30(tdx, ctx, n_w):
    import time

    import torch
    n_t, us = 300, []
    rng = np.random.default_rng(n_w)
    tr = tdx.Transitions(n_t, 0, paired=True)
    tr.delta.copy_(torch.from_numpy(rng.uniform(0.05, 1.5, n_t)))
    tr.df.copy_(torch.from_numpy(rng.uniform(0.1, 1.0, n_t)))
    om = torch.linspace(0.0, 2.0, n_w, device="cuda", dtype=torch.float64)
    P = torch.ones((n_t, 32), dtype=torch.complex64, device="cuda")
    for n_g in (29, 30):
        P[:, n_g:] = 0
        out = torch.empty(n_w * n_g * n_g, dtype=torch.complex128, device="cuda")
        best = 1e9
        for _ in range(20):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(20):
                tdx.chi0(ctx, tr, P, n_g, "fp32", om, ETA, PREF, out=out)
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - t0) / 20)
        us.append(1e6 * best)
        print("chi0 fp32 short", n_w, n_g, us, flush=True)
        P[:, :] = 1
    assert us[0] < 1.12 * us[1]
