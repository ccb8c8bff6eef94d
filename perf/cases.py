"""The work that programs have this framework do, as cases that can be timed.

Every case goes through the public calls of the binding.  The single steps
(spectra, attenuation, conductivity, Dyson, pair densities, chi0 and its
adjoint) take inputs that are made here from a seed; the whole calls (run_q,
the gradient) take a workload.  States are nearly free electrons on the
plane-wave spheres of the workload's cell: kinetic energies with a small
seeded potential, orbitals dominated by their own plane wave with tails that
fall with the energy distance, Fermi-Dirac occupations at the workload's
temperature.  They have the sizes, spectra and occupations of the crystal and
the electron gas without an eigensolve, whose cost a program pays once.

`exact` states the same results in 64 bits with plain torch.
"""
import math

import numpy as np
import torch

import paper_2510_01875_amd as tdx
import workloads
from paper_2510_01875_amd import grad

EV = 1.0 / 27.211386245988
THR = 1e-8          # |df| screening of every workload
ETA = 0.5 * EV      # broadening of the crystal workloads
C2 = workloads.fcc_c2()

_ctx = None


def ctx():
    """One context per process, as a program keeps it."""
    global _ctx
    if _ctx is None:
        _ctx = tdx.Context(0)
    return _ctx


# ------------------------------------------------------------------- cases
def listed():
    return [
        # the smallest calls: S, F, the imaginary-time metrics and the dielectric
        # properties of one q from its chi_00 on the crystal's 500 frequencies
        dict(name="spectra", kind="spectra", n_w=500, n_tau=65),
        # the Savitzky-Golay grid search on one spectrum: degrees 1-6, windows 5-61,
        # 86 (window, degree) pairs, the benchmark's search
        dict(name="attenuation", kind="attenuation", n_w=500, n_tau=65, win_lo=5, win_hi=61,
             win_step=4, deg_hi=6),
        # the Kubo-Greenwood route of the crystal at 4 eV: sigma of the states, S*, way back
        dict(name="conductivity", kind="conductivity", k=5, t_ev=4.0, n_w=499),
        # one crystal q's Dyson solves with the dense (ALDA) kernel
        dict(name="dyson", kind="dyson", n_g=133, n_w=500),
        # one crystal q's pair densities in FP64 (what the reverse sweep recomputes)
        dict(name="pair_density", kind="pair_density", k=5, t_ev=2.0, e_chi=8.5, j=1, prec="fp64",
             paired=True),
        # the chi0 contraction in FP64, the default precision, at the crystal's basis
        dict(name="chi0_fp64", kind="chi0", prec="fp64", n_g=133, n_w=500, n_t=50000, paired=True),
        # the same in FP32, at another of the crystal's bases
        dict(name="chi0_fp32", kind="chi0", prec="fp32", n_g=116, n_w=500, n_t=100000,
             paired=True),
        # a ragged batch of q in split-BF16: one persistent launch of a kept plan
        dict(name="chi0_batch", kind="chi0_batch", prec="bf16x3", n_q=4, n_g=116, n_w=500,
             n_t=40000),
        # a whole q of the electron gas (200 frequencies, RPA, FP64), the smallest workload
        dict(name="run_q_feg", kind="run_q", system="feg", k=8, t_ev=0.0, e_chi=2.0, j=8,
             n_w=200, prec="fp64"),
        # a whole q of the crystal (500 frequencies, ALDA, split-BF16) on a 5^3 grid
        dict(name="run_q_crystal", kind="run_q", system="fcc", k=5, t_ev=1.0, e_chi=8.5, j=1,
             n_w=500, prec="bf16x3"),
        # the chi0 step of the reverse sweep: one block of transitions with its
        # pair-density cotangents
        dict(name="chi0_vjp", kind="chi0_vjp", n_g=133, n_w=500, n_t=50000, paired=True),
        # value and gradient of F in T, eta and the shell values: 4 protons, two q
        dict(name="gradient", kind="gradient", n_w=120, k=2, e_wf=4.0, n_bands=64),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["spectra", "attenuation", "conductivity", "dyson", "pair_density", "chi0",
                       "chi0", "chi0_batch", "run_q", "chi0_vjp", "chi0_vjp", "dyson"])
    n_g = int(_log(rng, 17, 305))
    n_w = int(_log(rng, 40, 1001))
    flops = _log(rng, 2e10, 3.5e12)  # listed chi0_fp64: 3.5e12
    n_t = max(200, min(200000, int(flops / (8.0 * n_w * n_g * n_g))))
    if kind == "spectra":
        return dict(kind=kind, n_w=int(_log(rng, 40, 1001)), n_tau=2 * rng.randint(16, 64) + 1)
    if kind == "attenuation":
        return dict(kind=kind, n_w=int(_log(rng, 160, 1001)), n_tau=2 * rng.randint(16, 48) + 1,
                    win_lo=rng.choice([5, 9, 11]), win_hi=rng.randint(30, 75),
                    win_step=rng.choice([4, 6, 8]), deg_hi=rng.randint(2, 7))
    if kind == "conductivity":
        return dict(kind=kind, k=rng.randint(2, 5), t_ev=round(rng.uniform(0.8, 4.0), 3),
                    n_w=int(_log(rng, 40, 500)))
    if kind == "dyson":
        while n_g * n_g * n_w > 133 * 133 * 500:
            n_w = n_w * 3 // 4
        return dict(kind=kind, n_g=n_g, n_w=n_w)
    if kind == "pair_density":
        return dict(kind=kind, k=rng.randint(2, 5), t_ev=round(rng.uniform(0.8, 2.0), 3),
                    e_chi=round(rng.uniform(2.0, 8.5), 3), j=rng.randint(1, 2),
                    prec=rng.choice(["fp64", "fp64", "fp32"]), paired=rng.random() < 0.7)
    if kind == "chi0":
        return dict(kind=kind, prec=rng.choice(["fp64", "fp64", "fp32", "bf16x3"]), n_g=n_g,
                    n_w=n_w, n_t=n_t, paired=rng.random() < 0.7)
    if kind == "chi0_batch":
        return dict(kind=kind, prec=rng.choice(["bf16x3", "bf16x3", "fp64"]), n_q=rng.randint(2, 4),
                    n_g=int(_log(rng, 17, 140)), n_w=int(_log(rng, 40, 500)),
                    n_t=int(_log(rng, 500, 8000)))
    if kind == "run_q":
        if rng.random() < 0.5:
            return dict(kind=kind, system="feg", k=rng.choice([2, 3, 4, 6]), t_ev=0.0,
                        e_chi=round(rng.uniform(1.2, 2.4), 3), j=rng.randint(1, 6),
                        n_w=int(_log(rng, 40, 300)), prec=rng.choice(["fp64", "bf16x3"]))
        return dict(kind=kind, system="fcc", k=rng.randint(2, 4), t_ev=round(rng.uniform(0.8, 1.5), 3),
                    e_chi=round(rng.uniform(3.0, 8.5), 3), j=1, n_w=int(_log(rng, 40, 500)),
                    prec=rng.choice(["fp64", "bf16x3"]))
    n_t = max(200, min(50000, int(_log(rng, 1e8, 3.3e9) / (n_w * n_g))))
    return dict(kind="chi0_vjp", n_g=n_g, n_w=n_w, n_t=n_t, paired=rng.random() < 0.7)


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) + 7919)


def _cn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.complex128)


def _omega(n_w, top=2.0):
    return torch.linspace(0.0, top, n_w, dtype=torch.float64, device="cuda")


def _fermi(eps, nk, n_el, T):
    """Chemical potential and occupations of eps (numpy [n_k, nb]), two electrons a state."""
    lo, hi = eps.min() - 10 * T, eps.max() + 10 * T
    f = lambda mu: 0.5 * (1.0 - np.tanh(0.5 * (eps - mu) / T))  # noqa: E731
    for _ in range(200):
        mu = 0.5 * (lo + hi)
        if 2.0 / nk * f(mu).sum() < n_el:
            lo = mu
        else:
            hi = mu
    return mu, f(mu)


def _workload(case):
    k, n_w = case["k"], case.get("n_w", 500)
    if case.get("system", "fcc") == "feg":
        w = workloads.feg_c1()
        return w.with_(kgrid=(k, k, k), n_omega=n_w, qs=((case["j"], 0, 0),),
                       ecut_chi=(case["e_chi"],))
    j = case.get("j", 0)
    return C2.with_(kgrid=(k, k, k), n_omega=n_w, qs=((0, j, j),), temperatures=(case["t_ev"] * EV,),
                    ecut_chi=(case.get("e_chi", 8.5),), omega_max=(2.0,))


def _states(w, seed):
    """Nearly-free-electron states of a workload's sizes (see the file's head)."""
    g = _gen(seed)
    rng = np.random.default_rng(5)  # the levels, and so the list's length, are the system's own
    A = np.array(w.cell)
    B = 2 * math.pi * np.linalg.inv(A).T
    N = np.array(w.kgrid)
    nk = int(np.prod(N))
    span = int(math.sqrt(2 * w.ecut_wf) * np.linalg.norm(A, axis=1).max() / (2 * math.pi)) + 2
    ax = np.arange(-span, span + 1)
    M = np.stack(np.meshgrid(ax, ax, ax, indexing="ij"), -1).reshape(-1, 3)
    spheres = []
    for k in range(nk):
        r = np.array([k // (N[1] * N[2]), (k // N[2]) % N[1], k % N[2]])
        e = 0.5 * (((2 * r + 1 - N) / (2 * N) + M) @ B).__pow__(2).sum(1)
        keep = np.nonzero(e <= w.ecut_wf)[0]
        keep = keep[np.argsort(e[keep], kind="stable")]
        spheres.append((M[keep], e[keep]))
    npw = np.array([len(e) for _, e in spheres])
    d = tdx.StatesDims()
    d.n_k, d.npw_max, d.nb_max = nk, int(npw.max()), w.n_bands + 64
    st = tdx.States(d, 0)
    miller = np.zeros((nk, d.npw_max, 3), dtype=np.int32)
    kin = np.full((nk, d.npw_max), 1e3)
    eps = np.zeros((nk, w.n_bands))
    for k, (m, e) in enumerate(spheres):
        miller[k, :len(m)], kin[k, :len(m)] = m, e
        eps[k] = np.sort(e[:w.n_bands] + 0.02 * rng.standard_normal(w.n_bands))
    T = w.temperatures[0]
    mu, occ = _fermi(eps, nk, w.n_electrons, T)
    nb = w.n_bands
    st.npw.copy_(torch.from_numpy(npw.astype(np.int32)))
    st.nb.fill_(nb)
    st.miller.copy_(torch.from_numpy(miller))
    st.eps[:, :nb].copy_(torch.from_numpy(eps))
    st.occ[:, :nb].copy_(torch.from_numpy(occ))
    E = torch.from_numpy(kin).cuda()
    tail = 0.2 / (1.0 + 2.0 * (E[:, :nb, None] - E[:, None, :]).abs())
    tail = tail * (E[:, None, :] < 500.0)
    c = _cn(g, nk, nb, d.npw_max) * tail
    i = torch.arange(nb, device="cuda")
    c[:, i, i] += 1.0
    st.coef[:, :nb] = c / torch.linalg.vector_norm(c, dim=2, keepdim=True)
    s = st.c
    s.kgrid[:] = [int(x) for x in N]
    s.mmax[:] = [int(x) for x in np.abs(miller).max((0, 1))]
    s.cell[:] = list(A.reshape(-1))
    s.bvec[:] = list(B.reshape(-1))
    s.omega_cell = abs(float(np.linalg.det(A)))
    s.mu, s.temperature, s.beta = float(mu), T, 1.0 / T
    s.n_electrons = w.n_electrons
    s.density = w.n_electrons / s.omega_cell
    s.chi0_pref = 2.0 / (nk * s.omega_cell)
    return st


def _list(n_t, paired, g, T=2.0 * EV):
    """A transition list with the energies and occupation differences of a 3-electron gas."""
    u = torch.rand(2, n_t, generator=g, device="cuda", dtype=torch.float64)
    mu = 0.43
    e1 = (mu + 8 * T) * u[0] ** (2.0 / 3.0)
    e2 = 6.0 * u[1] ** (2.0 / 3.0)
    f = 0.5 * (1.0 - torch.tanh(0.5 * (torch.stack([e1, e2]) - mu) / T))
    tr = tdx.Transitions(n_t, 0, paired)
    tr.delta.copy_(e2 - e1)
    tr.df.copy_(f[0] - f[1])
    return tr


def _rho(n_t, n_g, g):
    """Pair densities [n_t, n_g]: amplitudes that fall with |q + G|."""
    amp = 0.3 * torch.exp(-3.0 * torch.arange(n_g, device="cuda", dtype=torch.float64) / n_g)
    return _cn(g, n_t, n_g) * amp


def _store(rho, prec):
    """rho in the layout of a precision (tdx.h, tdx_pair_density)."""
    n_t, n_g = rho.shape
    ld = (n_g + 15) // 16 * 16
    if prec != "bf16x3":
        P = torch.zeros((n_t, ld), dtype=torch.complex128 if prec == "fp64" else torch.complex64,
                        device="cuda")
        P[:, :n_g] = rho
        return torch.view_as_real(P).reshape(-1).view(torch.uint8)
    rows = ((n_t + 31) // 32 + 1) * 32
    x = torch.zeros((rows, ld, 2), dtype=torch.float32, device="cuda")
    x[:n_t, :n_g] = torch.view_as_real(rho).float()
    hi = x.to(torch.bfloat16)
    lo = (x - hi.float()).to(torch.bfloat16)
    frag = torch.stack([hi, lo]).view(2, rows // 4, 4, ld, 2).permute(1, 0, 3, 2, 4).contiguous()
    return torch.cat([frag.reshape(-1).view(torch.uint8), x.reshape(-1).view(torch.uint8)])


def _batch_sizes(case):
    """(n_g, n_w, n_t) of a batch's items: bases and lists that differ from q to q."""
    return [(case["n_g"] + (0, 17, 35, 13)[i], case["n_w"] + (0, 0, 37, 11)[i],
             case["n_t"] * (1, 2, 1, 3)[i] + 5 * i) for i in range(case["n_q"])]


def _chi0_inputs(n_g, n_t, paired, seed):
    g = _gen(seed)
    return _list(n_t, paired, g), _rho(n_t, n_g, g)


def _dyson_inputs(n_g, n_w, seed):
    """chi0(w) = H_R + i H_A of a few hundred transitions and K = v + a small Hermitian part."""
    g = _gen(seed)
    om = _omega(n_w)
    tr, rho = _list(2 * n_g + 100, True, g), _rho(2 * n_g + 100, n_g, g)
    chi0 = _exact_chi0(tr.delta, tr.df, True, rho, om, ETA, 6.0 / len(tr))
    q2 = torch.linspace(0.5, 17.0, n_g, dtype=torch.float64, device="cuda")
    h = _cn(g, n_g, n_g)
    K = torch.diag(4 * math.pi / q2).to(torch.complex128) - 0.05 * (h + h.mH) / 2
    return om, chi0, K, n_g // 3


def _spectrum_inputs(case, seed):
    rng = np.random.default_rng(seed)
    om = np.linspace(0.0, 2.0, case["n_w"])
    w0, gam = 0.5 + 0.2 * rng.random(3), 0.05 + 0.1 * rng.random(3)
    chi = sum(a / (om ** 2 - x * x + 1j * y * om) for a, x, y in zip((0.02, 0.01, 0.005), w0, gam))
    beta = 1.0 / ((1.0 + rng.random()) * EV)
    tau = np.linspace(0.0, beta, case["n_tau"])
    return om, chi, beta, tau


def prepare(case, seed):
    kind, g = case["kind"], _gen(seed)
    up = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    s = dict(kind=kind, ctx=ctx(), case=case)
    if kind == "spectra":
        om, chi, beta, tau = _spectrum_inputs(case, seed)
        s.update(om=up(om), chi=up(chi), beta=beta, tau=up(tau))
    elif kind == "attenuation":
        om, S, nu = workloads.rippled_spectrum(seed=seed, n_w=case["n_w"])
        beta = 1.0 / EV
        win, deg = _filters(case)
        s.update(om=up(om), S=up(S), nu=up(nu), beta=beta, win=win, deg=deg,
                 tau=up(np.linspace(0.0, beta, case["n_tau"])))
    elif kind == "conductivity":
        w = _workload(case)
        st = _states(w, seed)
        tr = tdx.transitions(s["ctx"], st, (0, 0, 0), THR)
        om = _omega(case["n_w"] + 1)[1:].contiguous()
        work = torch.empty(tdx.kg_work_bytes(len(tr), case["n_w"]), dtype=torch.uint8, device="cuda")
        s.update(st=st, tr=tr, om=om, work=work)
    elif kind == "dyson":
        om, chi0, K, i_g0 = _dyson_inputs(case["n_g"], case["n_w"], seed)
        s.update(chi0=chi0, K=K, i_g0=i_g0)
    elif kind == "pair_density":
        w = _workload(case)
        st = _states(w, seed)
        basis, _ = tdx.response_basis(w.cell, w.kgrid, w.qs[0], w.ecut_chi[0])
        tr = tdx.transitions(s["ctx"], st, w.qs[0], THR, paired=case["paired"])
        P = torch.empty(tdx.pair_density_bytes(len(tr), len(basis), case["prec"]),
                        dtype=torch.uint8, device="cuda")
        s.update(st=st, qj=w.qs[0], gb=torch.from_numpy(basis).cuda(), tr=tr, P=P)
    elif kind == "chi0":
        tr, rho = _chi0_inputs(case["n_g"], case["n_t"], case["paired"], seed)
        s.update(tr=tr, P=_store(rho, case["prec"]), om=_omega(case["n_w"]))
    elif kind == "chi0_batch":
        items = []
        for i, (n_g, n_w, n_t) in enumerate(_batch_sizes(case)):
            tr, rho = _chi0_inputs(n_g, n_t, True, 10 * seed + i)
            items.append(tdx.Chi0Item(tr, _store(rho, case["prec"]), n_g, _omega(n_w), ETA, 1e-4))
        s.update(plan=tdx.Chi0Plan(s["ctx"], items, case["prec"]))
    elif kind == "run_q":
        w = _workload(case)
        s.update(w=w, st=_states(w, seed))
    elif kind == "chi0_vjp":
        tr, rho = _chi0_inputs(case["n_g"], case["n_t"], case["paired"], seed)
        s.update(tr=tr, P=_store(rho, "fp64"), om=_omega(case["n_w"]), u=_cn(g, case["n_w"], case["n_g"]),
                 v=_cn(g, case["n_w"], case["n_g"]))
    else:
        k = case["k"]
        w = workloads.h_tiny(seed).with_(kgrid=(k, k, k), n_omega=case["n_w"], ecut_wf=case["e_wf"],
                                         n_bands=case["n_bands"], qs=((k, 0, 0), (1, 1, 0)))
        cot = torch.randn(2, w.n_tau, generator=g, device="cuda", dtype=torch.float64)
        s.update(w=w, cot=cot, runner=grad.ChainRunner(s["ctx"], w))
    return s


def _filters(case):
    pairs = [(x, d) for d in range(1, case["deg_hi"] + 1)
             for x in range(case["win_lo"], case["win_hi"] + 1, case["win_step"]) if x > d + 2]
    return [x for x, _ in pairs], [d for _, d in pairs]


DENSITY, Q2 = 0.027, 0.33   # electron density of the crystal, |q|^2 of its first q


def run(s):
    c, kind, case = s["ctx"], s["kind"], s["case"]
    if kind == "spectra":
        S = tdx.dsf(c, s["chi"], s["om"], s["beta"], DENSITY)
        F = tdx.itcf(c, S, s["om"], s["beta"], s["tau"])
        m = tdx.itcf_metrics(c, F, s["tau"], s["beta"], DENSITY)
        chi, eps_inv, sigma = tdx.dielectric(c, S, s["om"], s["beta"], DENSITY, Q2)
        return dict(S=S, F=F, metrics=m, chi=chi, eps_inv=eps_inv, sigma=sigma)
    if kind == "attenuation":
        a = tdx.attenuate(c, s["S"], s["om"], s["beta"], s["tau"], s["win"], s["deg"], s["nu"])
        return dict(Sp=a.Sp, scores=a.scores, resid=a.resid, best=[a.best[d] for d in sorted(a.best)])
    if kind == "conductivity":
        sig = tdx.kg_conductivity(c, s["st"], s["om"], ETA, THR, tr=s["tr"], work=s["work"])
        st = s["st"]
        S = tdx.kg_dsf(c, sig, s["om"], st.beta, st.density)
        chi, eps_inv, back = tdx.kg_dielectric(c, S, s["om"], st.beta, st.density)
        return dict(sigma=sig, S=S, chi=chi, eps_inv=eps_inv, back=back)
    if kind == "dyson":
        return tdx.dyson(c, s["chi0"], s["K"], s["i_g0"])
    if kind == "pair_density":
        P = tdx.pair_density(c, s["st"], s["qj"], s["tr"], s["gb"], case["prec"], out=s["P"])
        return tdx.pair_density_view(P, len(s["tr"]), s["gb"].shape[0], case["prec"])
    if kind == "chi0":
        return tdx.chi0(c, s["tr"], s["P"], case["n_g"], case["prec"], s["om"], ETA, 1e-4)
    if kind == "chi0_batch":
        s["plan"].launch()
        return [it.out for it in s["plan"].items]
    if kind == "run_q":
        q = tdx.run_q(c, s["w"], s["st"], 0, case["prec"])
        return dict(chi0=q.chi0, K=q.K, chi00=q.chi00, S=q.S, F=q.F, n_trans=q.n_trans)
    if kind == "chi0_vjp":
        w_bar, rho_bar = tdx.chi0_vjp(c, s["tr"], s["P"], case["n_g"], s["om"], ETA, 1e-4, s["u"],
                                      s["v"], want_rho=True)
        return dict(w_bar=w_bar, rho_bar=rho_bar[:, :case["n_g"]])
    w = s["w"]
    T = torch.tensor(w.temperatures[0], dtype=torch.float64, requires_grad=True)
    eta = torch.tensor(w.eta, dtype=torch.float64, requires_grad=True)
    v = torch.tensor(w.potential.shell_v, dtype=torch.float64, requires_grad=True)
    F = grad.itcf_differentiable(c, w, T, eta, v, s["runner"])
    (F * s["cot"]).sum().backward()
    return dict(F=F.detach(), T=T.grad, eta=eta.grad, v=v.grad)


# -------------------------------------------------------------------- work
def _run_sizes(case):
    """(n_trans, n_g, npw, nb, n_k) of a crystal or electron-gas case, estimated from its sizes:
    the occupation window sets the occupied bands that every other band pairs with."""
    w = _workload(case)
    nk = w.n_k
    vol = abs(float(np.linalg.det(np.array(w.cell))))
    sphere = lambda e: (2 * e) ** 1.5 * vol / (6 * math.pi ** 2)  # noqa: E731
    T = w.temperatures[0]
    n = w.n_electrons / vol
    top = max(0.5 * (3 * math.pi ** 2 * n) ** (2.0 / 3.0), 0.0) + 18.0 * T  # f > THR
    occ = min(w.n_bands, max(1.0, sphere(top)))
    full = nk * (2 * occ * w.n_bands - occ * occ)
    return full, max(1.0, sphere(w.ecut_chi[0])), sphere(w.ecut_wf), w.n_bands, nk


def work(case):
    kind = case["kind"]
    n_w, n_g = case.get("n_w", 0), case.get("n_g", 0)
    if kind == "spectra":
        n_tau = case["n_tau"]
        # chi00, omega, tau in; S, F, metrics, chi, eps^-1, sigma out
        return dict(bytes=8.0 * (12 * n_w + 3 * n_tau), flops=n_w * (60.0 * n_tau + 60.0 * n_w))
    if kind == "attenuation":
        win, deg = _filters(case)
        fl = sum(2.0 * x * (d + 1) for x, d in zip(win, deg)) * n_w + len(win) * n_w * 60.0 * case["n_tau"]
        return dict(bytes=8.0 * n_w * (3 + 2 * len(win)), flops=fl)
    if kind == "conductivity":
        full, _, npw, nb, nk = _run_sizes(case)
        return dict(bytes=16.0 * nk * nb * npw + 32.0 * full, flops=full * (20.0 * npw + 10.0 * n_w))
    if kind == "dyson":
        # 1 - chi0 K and its LU
        return dict(bytes=16.0 * n_g * n_g * (n_w + 1), flops=n_w * (8.0 + 8.0 / 3.0) * n_g ** 3)
    if kind == "pair_density":
        full, ng, npw, nb, nk = _run_sizes(case)
        t = full / 2 if case["paired"] else full
        size = 16 if case["prec"] == "fp64" else 8
        return dict(bytes=16.0 * nk * nb * npw + t * ng * size, flops=8.0 * t * ng * npw)
    size = {"fp64": 16, "fp32": 8, "bf16x3": 16}.get(case.get("prec"), 16)
    if kind == "chi0":
        # one product per real component of rho rho^H (n_g^2 of them) and part of w
        return dict(bytes=case["n_t"] * (n_g * size + 16.0) + 16.0 * n_w * n_g * n_g,
                    flops=4.0 * n_w * n_g * n_g * case["n_t"])
    if kind == "chi0_batch":
        z = _batch_sizes(case)
        return dict(bytes=sum(t * (g * size + 16.0) + 16.0 * w * g * g for g, w, t in z),
                    flops=sum(4.0 * w * g * g * t for g, w, t in z))
    if kind == "run_q":
        full, ng, npw, nb, nk = _run_sizes(case)
        t = full / 2
        return dict(bytes=16.0 * nk * nb * npw + 16.0 * n_w * ng * ng,
                    flops=t * ng * (8.0 * npw + 4.0 * n_w * ng) + n_w * 10.7 * ng ** 3)
    if kind == "chi0_vjp":
        # u^H rho, v^H rho and the cotangent's two products
        return dict(bytes=32.0 * case["n_t"] * n_g + 32.0 * n_w * n_g, flops=32.0 * case["n_t"] * n_w * n_g)
    k3, vol = case["k"] ** 3, 4.0 / workloads.paper_h_density()
    npw = (2 * case["e_wf"]) ** 1.5 * vol / (6 * math.pi ** 2)
    t = k3 * case["n_bands"] ** 2 / 2.0
    return dict(bytes=16.0 * k3 * case["n_bands"] * npw * 3,
                flops=2 * t * 40 * (24.0 * npw + 32.0 * n_w) + k3 * 40.0 * npw ** 3)


# ------------------------------------------------------------------- exact
def _weights(delta, df, paired, om, eta):
    z = om[:, None] + 1j * eta
    if paired:
        return 2.0 * df * delta / (z * z - delta * delta)
    return df / (z - delta)


def _exact_chi0(delta, df, paired, rho, om, eta, pref):
    n_g = rho.shape[1]
    out = torch.zeros((om.shape[0], n_g * n_g), dtype=torch.complex128, device="cuda")
    step = max(64, min(4096, (1 << 25) // (n_g * n_g)))
    for b in range(0, rho.shape[0], step):
        r = rho[b:b + step]
        X = (r[:, :, None] * r.conj()[:, None, :]).reshape(r.shape[0], -1)
        out += _weights(delta[b:b + step], df[b:b + step], paired, om, eta) @ X
    return (pref * out).view(-1, n_g, n_g)


def _exact_pairs(w, st, qj, basis, paired):
    """(delta, df, rho [T, n_g]) of the states' screened list, k by k from the definition."""
    N = np.array(w.kgrid)
    nk, nb = w.n_k, w.n_bands
    npw, mil = st.npw.cpu().numpy(), st.miller.cpu().numpy()
    big = int(np.abs(mil).max()) + int(np.abs(basis).max()) + int(max(abs(x) for x in qj)) + 2
    side = 2 * big + 1
    out = []
    for k in range(nk):
        r = np.array([k // (N[1] * N[2]), (k // N[2]) % N[1], k % N[2]])
        s = r + np.array(qj)
        r2 = s % N
        gs = (s - r2) // N
        k2 = int((r2[0] * N[1] + r2[1]) * N[2] + r2[2])
        rt = (N - 1 - r - np.array(qj)) % N
        kt = int((rt[0] * N[1] + rt[1]) * N[2] + rt[2])
        if paired and kt < k:
            continue
        df = st.occ[k, :nb, None] - st.occ[k2, None, :nb]
        hit = df.abs() > THR
        if paired and kt == k:
            hit = hit & torch.ones(nb, nb, dtype=torch.bool, device="cuda").triu(1)
        n, m = torch.nonzero(hit, as_tuple=True)
        if not n.numel():
            continue
        box = np.full((side, side, side), -1, dtype=np.int64)
        m2 = mil[k2, :npw[k2]] + big
        box[m2[:, 0], m2[:, 1], m2[:, 2]] = np.arange(npw[k2])
        x = mil[k, :npw[k]][None] + basis[:, None] + gs + big
        x = np.clip(x, 0, side - 1)  # the rim of the box holds no plane wave
        idx = torch.from_numpy(box[x[..., 0], x[..., 1], x[..., 2]]).cuda()
        a = st.coef[k, :nb, :npw[k]].conj()
        b = st.coef[k2, :nb]
        rho = torch.empty((n.numel(), len(basis)), dtype=torch.complex128, device="cuda")
        for g in range(len(basis)):
            bg = b[:, idx[g].clamp(min=0)] * (idx[g] >= 0)
            rho[:, g] = (a @ bg.T.contiguous())[n, m]
        out.append((st.eps[k2, m] - st.eps[k, n], df[n, m], rho))
    return [torch.cat(x) for x in zip(*out)]


def _exact_dsf(chi00, om, beta, dens):
    S = -chi00.imag / (math.pi * dens * -torch.expm1(-beta * om))
    if om[0] == 0.0:
        S[0] = -chi00.imag[1] / (math.pi * dens * beta * om[1])
    return S


def _trapezoid(x):
    c = torch.zeros_like(x)
    c[1:] += 0.5 * (x[1:] - x[:-1])
    c[:-1] += 0.5 * (x[1:] - x[:-1])
    return c


def _exact_itcf(S, om, beta, tau):
    e = torch.exp(-tau[:, None] * om) + torch.exp(-(beta - tau)[:, None] * om)
    return (S[..., None, :] * (_trapezoid(om) * e)).sum(-1)


def _exact_dielectric(S, om, beta, dens, q2):
    im = math.pi * dens * torch.expm1(-beta * om) * S
    a, b, fa, fb = om[:-1], om[1:], im[:-1], im[1:]
    sl = (fb - fa) / (b - a)
    re = (2.0 * sl * (b - a)).sum().expand_as(om)
    for c in (om[:, None], -om[:, None]):
        lg = lambda x: torch.where(x == 0, 0.0, x.abs().clamp(min=1e-300).log())  # noqa: E731
        re = re + ((fa + sl * (c - a)) * (lg(b - c) - lg(a - c))).sum(1)
    chi = torch.complex(re / math.pi, im)
    eps_inv = 1.0 + 4 * math.pi / q2 * chi
    return chi, eps_inv, -1j * om * (1.0 / eps_inv - 1.0) / (4 * math.pi)


def _exact_attenuation(case, s):
    S, om, n = s["S"].cpu().numpy(), s["om"], case["n_w"]
    Sp = np.empty((len(s["win"]), n))
    k = np.empty(len(s["win"]))
    for f, (x, d) in enumerate(zip(s["win"], s["deg"])):
        Q, _ = np.linalg.qr(np.vander(np.linspace(-1, 1, x), d + 1, increasing=True))
        H = Q @ Q.T
        at = np.clip(np.arange(n) - x // 2, 0, n - x)
        rows = H[np.arange(n) - at]
        Sp[f] = (rows * S[at[:, None] + np.arange(x)]).sum(1)
        k[f] = H.diagonal()[np.arange(n) - at].sum()
    Sp = torch.from_numpy(Sp).cuda()
    S, k = s["S"], torch.from_numpy(k).cuda()
    rss = ((Sp - S) ** 2).sum(1)
    aicc = n * torch.log(rss / n) + 2 * k + 2 * k * (k + 1) / (n - k - 1)
    D = lambda y: (y[..., 2:] - y[..., :-2]) / (om[2:] - om[:-2])  # noqa: E731
    ph = torch.exp(-2j * math.pi * s["nu"][:, None] * om[1:-1])
    power = lambda y: (D(y)[..., None, :] * ph).mean(-1).abs() ** 2  # noqa: E731
    curv = lambda y: (torch.diff(y, n=2) ** 2).sum(-1)  # noqa: E731
    scores = torch.stack([rss, k, aicc, (power(Sp) / power(S)).mean(1), curv(Sp) / curv(S)], 1)
    beta, tau = s["beta"], s["tau"]
    F, Fp = _exact_itcf(S, om, beta, tau), _exact_itcf(Sp, om, beta, tau)
    R, c, mid = F - Fp, _trapezoid(tau) / beta, F[case["n_tau"] // 2]
    mean = (R * c).sum(1)
    sig = torch.sqrt((((R - mean[:, None]) ** 2) * c).sum(1))
    resid = torch.stack([(R / F).abs().max(1).values, mean / mid, sig / mid], 1)
    return dict(Sp=Sp, scores=scores, resid=resid, best=None)


def _exact_vjp(case, s, rho):
    om, u, v, tr = s["om"], s["u"], s["v"], s["tr"]
    d, f, pref = tr.delta, tr.df, 1e-4
    al, be = u.conj() @ rho.T.contiguous(), v.conj() @ rho.T.contiguous()
    z = om[:, None] + 1j * ETA
    r1, r2 = 1.0 / (z - d), 1.0 / (z + d)
    gw, hw, ew = (r1 - r2, r1 * r1 + r2 * r2, r1 * r1 - r2 * r2) if case["paired"] else (r1, r1 * r1, r1 * r1)
    lam = pref * al * be.conj()
    wb = torch.stack([(lam * gw).real.sum(0), f * (lam * hw).real.sum(0), f * (lam * ew).imag.sum(0)], 1)
    w = pref * f * gw
    rb = (w * be.conj()).conj().T.contiguous() @ u + (w * al).T.contiguous() @ v
    return dict(w_bar=wb, rho_bar=rb)


def exact(case, seed):
    kind = case["kind"]
    if kind == "gradient":
        return None
    s = prepare(case, seed) if kind in ("spectra", "attenuation") else {}
    if kind == "spectra":
        S = _exact_dsf(s["chi"], s["om"], s["beta"], DENSITY)
        tau, F = s["tau"], _exact_itcf(S, s["om"], s["beta"], s["tau"])
        A, mid = (F * _trapezoid(tau)).sum(), F[case["n_tau"] // 2]
        m = torch.stack([mid, A, mid - F[0], A - s["beta"] * F[0], -DENSITY * A])[None]
        chi, eps_inv, sigma = _exact_dielectric(S, s["om"], s["beta"], DENSITY, Q2)
        return dict(S=S, F=F, metrics=m, chi=chi, eps_inv=eps_inv, sigma=sigma)
    if kind == "attenuation":
        return _exact_attenuation(case, s)
    if kind == "dyson":
        _, chi0, K, i = _dyson_inputs(case["n_g"], case["n_w"], seed)
        c, K = chi0.cpu().numpy(), K.cpu().numpy()
        x = np.linalg.solve(np.eye(case["n_g"]) - c @ K, c[:, :, i:i + 1])
        return torch.from_numpy(x[:, i, 0].copy())
    if kind in ("chi0", "chi0_batch"):
        out = []
        z = [(case["n_g"], case["n_w"], case["n_t"])] if kind == "chi0" else _batch_sizes(case)
        for i, (n_g, n_w, n_t) in enumerate(z):
            paired = case.get("paired", True)
            tr, rho = _chi0_inputs(n_g, n_t, paired, seed if kind == "chi0" else 10 * seed + i)
            if case["prec"] != "fp64":
                rho = rho.to(torch.complex64).to(torch.complex128)
            out.append(_exact_chi0(tr.delta, tr.df, paired, rho, _omega(n_w), ETA, 1e-4))
        return out[0] if kind == "chi0" else out
    if kind == "chi0_vjp":
        tr, rho = _chi0_inputs(case["n_g"], case["n_t"], case["paired"], seed)
        g = _gen(seed)
        u, v = _cn(g, case["n_w"], case["n_g"]), _cn(g, case["n_w"], case["n_g"])
        return _exact_vjp(case, dict(om=_omega(case["n_w"]), u=u, v=v, tr=tr), rho)
    w = _workload(case)
    st = _states(w, seed)
    if kind == "conductivity":
        return _exact_conductivity(case, w, st)
    # the order of B(q)'s vectors, a labelling that every call takes or returns
    basis, i_g0 = tdx.response_basis(w.cell, w.kgrid, w.qs[0], w.ecut_chi[0])
    paired = case.get("paired", True)
    delta, df, rho = _exact_pairs(w, st, w.qs[0], basis, paired)
    if kind == "pair_density":
        return rho if case["prec"] == "fp64" else rho.to(torch.complex64)
    om = _omega(case["n_w"])
    pref = 2.0 / (w.n_k * st.c.omega_cell)
    chi0 = _exact_chi0(delta, df, True, rho, om, w.eta, pref)
    if w.xc != "rpa":
        return dict(chi0=chi0, K=None, chi00=None, S=None, F=None, n_trans=None)
    B = np.array(list(st.c.bvec)).reshape(3, 3)
    qg = (np.array(w.qs[0]) / np.array(w.kgrid) + basis) @ B
    K = np.diag(4 * math.pi / (qg ** 2).sum(1)).astype(np.complex128)
    c = chi0.cpu().numpy()
    x = np.linalg.solve(np.eye(len(basis)) - c @ K, c[:, :, i_g0:i_g0 + 1])[:, i_g0, 0]
    chi00, beta = torch.from_numpy(x.copy()).cuda(), st.c.beta
    S = _exact_dsf(chi00, om, beta, st.c.density)
    F = _exact_itcf(S, om, beta, torch.from_numpy(w.tau_grid(0)).cuda())
    return dict(chi0=chi0, K=torch.from_numpy(K), chi00=chi00, S=S, F=F, n_trans=None)


def _exact_conductivity(case, w, st):
    om = _omega(case["n_w"] + 1)[1:]
    B = torch.tensor(list(st.c.bvec), dtype=torch.float64, device="cuda").view(3, 3)
    N = np.array(w.kgrid)
    nb = w.n_bands
    sig = torch.zeros_like(om).to(torch.complex128)
    for k in range(w.n_k):
        r = np.array([k // (N[1] * N[2]), (k // N[2]) % N[1], k % N[2]])
        kr = torch.from_numpy((2 * r + 1 - N) / (2 * N)).cuda()
        npw = int(st.npw[k])
        G = (kr + st.miller[k, :npw].double()) @ B
        c = st.coef[k, :nb, :npw]
        p2 = sum(((c.conj() * G[:, a]) @ c.T.contiguous()).abs() ** 2 for a in range(3))  # [m, n]
        df = st.occ[k, :nb, None] - st.occ[k, None, :nb]
        n, m = torch.nonzero(df.abs() > THR, as_tuple=True)
        d = st.eps[k, m] - st.eps[k, n]
        W = df[n, m] / d * p2[m, n] / 3.0
        for b in range(0, n.numel(), 1 << 16):
            z = om[:, None] - d[None, b:b + (1 << 16)] + 1j * ETA
            sig += (W[b:b + (1 << 16)] / z).sum(1)
    sig = 2j / (st.c.omega_cell * w.n_k) * sig
    eps = 1.0 + 4j * math.pi * sig / om
    beta, dens = st.c.beta, st.c.density
    S = _exact_dsf(1.0 / eps - 1.0, om, beta, dens)
    chi, eps_inv, back = _exact_dielectric(S, om, beta, dens, 4 * math.pi)
    return dict(sigma=sig, S=S, chi=chi, eps_inv=eps_inv, back=back)
