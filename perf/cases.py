"""The work that a phaseless-AFQMC program has this framework do, as timed cases.

A case is one pass through the public entry points at one shape: whole steps of
the driver, and the step's parts as a program calls them one at a time.  The
kinds, and what each stands for:

  step     driver.step: one whole AFQMC step of a walker population
  energy   the mixed estimator's measurement: Green's functions of every path,
           then the Cholesky contraction to local energies and force bias
  move     one walker move: propagation with the phaseless weight, then the
           periodic re-orthonormalisation
  paths    Metropolis sweeps of every tethered path, then the hand-off
  trial    the sampled trial rebuilt from its hidden variables and measured
           (what a measurement with fresh paths does), multi-slice trials
  density  the back-propagated one-body density matrix

listed() has the shapes of the repository's own workloads (tiny, FP64, mixed,
learned, slices, and three of the uneven batch's shapes); draw() spreads the
same kinds over the sizes that afqmc_create takes.  Inputs are made by plain
torch and numpy from the seed alone; exact() gives the same quantities in 64
bits without this repository's code.
"""
import math

import numpy as np
import torch

import afqmc_inputs as ai
from paper_2505_18519_amd import afqmc as A
from paper_2505_18519_amd import driver as D

C128, F64 = torch.complex128, torch.float64
TAYLOR = 10          # Taylor order of exp(V)
TAU_T, SLICES = 0.01, 2

_DEFAULTS = dict(prec=0, c64=0, ising=0, slices=0, learned=0, sweeps=1, h=0)


def _case(kind, M, N, G, K, nw, P, name=None, **kw):
    c = dict(kind=kind, M=M, N=N, G=G, K=K, nw=nw, P=P, **_DEFAULTS)
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest population: the tiny Ising workload, one whole step; launches and
        # latency are all there is
        _case("step", 8, 2, 16, 4, 64, 8, name="step-tiny", ising=1),
        # the FP64 benchmark workload, one whole step of 512 walkers x 8 paths
        _case("step", 64, 16, 256, 64, 512, 8, name="step-m64"),
        # a ragged small system of an uneven batch (N = M/4, 4M vectors): orbitals and
        # electrons off every tile edge
        _case("energy", 45, 11, 180, 22, 333, 4, name="energy-m45"),
        # the learned workload's system measured in FP64 (its random-walk leg)
        _case("energy", 96, 24, 384, 128, 512, 4, name="energy-m96"),
        # one of the uneven batch's systems past M = 128 and N = 32
        _case("energy", 142, 35, 568, 71, 150, 4, name="energy-m142"),
        # the learned workload's measurement: FP32 products, full population
        _case("energy", 96, 24, 384, 128, 2048, 4, name="energy-fp32-m96", prec=1, c64=1),
        # the mixed workload's measurement: BF16 products, full population
        _case("energy", 128, 32, 512, 128, 1024, 4, name="energy-bf16-m128", prec=2, c64=1),
        # a ragged mid-sized system of an uneven batch: the walkers' move
        _case("move", 72, 18, 288, 36, 700, 4, name="move-m72"),
        # the FP64 workload's path updates at the several sweeps per step that the
        # converged energies need
        _case("paths", 64, 16, 256, 64, 512, 8, name="paths-m64", sweeps=4),
        # the learned proposal with the network training on the chains' own moves
        _case("paths", 96, 24, 384, 128, 512, 4, name="paths-learned-m96", prec=1, learned=1),
        # the multi-slice (complex) trial rebuilt from its fields and measured
        _case("trial", 64, 16, 256, 512, 256, 8, name="trial-slices-m64", slices=SLICES),
        # a back-propagated density matrix twenty steps deep
        _case("density", 64, 16, 256, 64, 128, 8, name="density-m64", h=20),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "energy", "energy", "energy", "move", "move", "paths", "paths",
                       "trial", "density"])
    kw = {}
    prec = rng.choice([0, 0, 0, 1, 2, 3]) if kind in ("step", "energy", "move", "paths") else 0
    top = 160 if prec == 0 and kind in ("energy", "move", "paths") else 128
    if kind in ("step", "density"):
        top = 96
    if kind == "trial":
        top = 80
    M = _log(rng, 8, top)
    # closed-shell fillings from an eighth to a third of the orbitals
    N = max(1, min(int(round(M * rng.uniform(0.125, 0.34))), 40 if top == 160 else 32))
    if kind == "trial":  # the complex trial's own size limit
        N = min(N, 16)
    G = max(4, int(round(M * rng.uniform(2.0, 4.5))))
    K = max(2, int(round(M * rng.uniform(0.4, 1.0))))
    P = rng.choice([1, 2, 3, 4, 4, 5, 8, 8, 12])
    nw = _log(rng, 8, 1500)
    if prec:
        kw.update(prec=prec, c64=rng.choice([0, 1]))
    if kind == "step" and prec == 0 and rng.random() < 0.2:
        kw.update(ising=1)
        K = min(K, 8)  # a sweep flips the variables one after another
    if kind == "paths":
        kw.update(sweeps=rng.choice([1, 2, 3]))
        if M <= 128 and N <= 32 and rng.random() < 0.25:
            kw.update(learned=1, prec=1, c64=0, sweeps=1)
    if kind == "trial":
        m = rng.choice([1, 2, 3])
        kw.update(slices=m)
        K = m * G
    if kind == "density":
        kw.update(h=rng.choice([0, 3, 8, 16]))
    # no dearer than the largest listed cases: bounded arithmetic and bounded state
    limit = 2.5e11 if kw.get("prec", 0) == 0 else 8e11
    c = _case(kind, M, N, G, K, nw, P, **kw)
    while nw > 1 and (work(c)["flops"] > limit or nw * P * M * M > 2.5e7):
        nw = max(1, int(nw * 0.8))
        c["nw"] = nw
    return c


# ---------------------------------------------------------------------------
# inputs: plain torch and numpy, from the seed alone


def _sym(u):
    u = torch.triu(u)
    return u + torch.triu(u, 1).transpose(-1, -2)


def _system(case, gen):
    """A Hamiltonian and trial of the shapes and value distributions of the
    repository's synthetic systems, as (System on the host, device arrays)."""
    M, N, G, K = case["M"], case["N"], case["G"], case["K"]
    z = dict(generator=gen, device="cuda", dtype=F64)
    h1 = torch.triu(0.1 * torch.randn(M, M, **z), 1)
    h1 = h1 + h1.T + torch.diag(torch.linspace(-2.0, 2.0, M, device="cuda", dtype=F64))
    scale = 0.3 * math.sqrt(8.0 / M) / torch.sqrt(torch.arange(1, G + 1, device="cuda", dtype=F64))
    L = _sym(torch.randn(G, M, M, **z) * scale[:, None, None]).contiguous()
    h1n = h1.cpu().numpy()
    lam, vec = np.linalg.eigh(h1n)
    sign = np.sign(vec[np.abs(vec).argmax(0), np.arange(M)])
    phi0 = np.ascontiguousarray((vec * sign)[:, :N])
    kw = {}
    if case["slices"]:
        m = case["slices"]
        Agen, kind, coupling = L, ai.HIDDEN_GAUSS, 0.0
        half = (vec * np.exp(-0.5 * TAU_T * lam)) @ vec.T
        full = (vec * np.exp(-TAU_T * lam)) @ vec.T
        F = np.stack([half] + [full] * (m - 1) + [half])
        kw = dict(trial_kind=ai.TRIAL_SLICES, n_slices=m, slice_s=np.full(m, TAU_T), slice_F=F)
    elif case["ising"]:
        kind, coupling = ai.HIDDEN_ISING, 0.2
        Agen = torch.zeros(K, M, M, device="cuda", dtype=F64)
        for k in range(K):
            for j in (2 * k % M, (2 * k + 1) % M):
                Agen[k, j, j] = 1.0
    else:
        kind, coupling = ai.HIDDEN_GAUSS, 0.1
        mask = torch.rand(K, M, M, **z) < 0.05
        Agen = _sym(torch.where(mask, torch.randn(K, M, M, **z), 0.0)).contiguous()
    Eh = (vec * np.exp(-0.5 * _dtau(case) * lam)) @ vec.T
    s = ai.System(M=M, N=N, n_chol=G, K=K, hidden_kind=kind, coupling=coupling, h1=h1n,
                  L=L.cpu().numpy(), phi0=phi0, A=Agen.cpu().numpy(), **kw)
    dev = dict(h1=h1, L=L, A=Agen, phi0=torch.from_numpy(phi0).cuda(),
               Eh=torch.from_numpy(np.ascontiguousarray(Eh)).cuda())
    return s, dev


def _dtau(case):
    return 0.01 if case["M"] <= 8 else 0.005


def _expm_apply(U, X):
    """exp(U) X for batches of symmetric U: scaled Taylor series, 64 bits."""
    norm = float(U.abs().sum(-1).max()) if U.numel() else 0.0
    parts = max(1, math.ceil(norm / 4.0))
    X = X.expand(U.shape[0], -1, -1).contiguous()
    for _ in range(parts):
        term, acc = X, X.clone()
        for j in range(1, 33):
            term = torch.bmm(U, term) / (parts * j)
            acc += term
        X = acc
    return X


def _taylor(V, X, order=TAYLOR):
    """T_order(V) X, complex, batches."""
    term, acc = X, X.clone()
    for j in range(1, order + 1):
        term = torch.bmm(V, term) / j
        acc = acc + term
    return acc


def _trial(case, s, dev, y):
    """Phi_T(y) [S, M, N] of the paths y [S, K]."""
    S, M = y.shape[0], case["M"]
    if not case["slices"]:
        U = s.coupling * (y @ dev["A"].reshape(case["K"], M * M)).reshape(S, M, M)
        return _expm_apply(U, dev["phi0"])
    m = case["slices"]
    F = torch.from_numpy(np.ascontiguousarray(s.slice_F)).cuda().to(C128)
    X = (F[0] @ dev["phi0"].to(C128)).expand(S, -1, -1)
    yl = y.reshape(S, m, case["G"])
    for l in range(m):
        V = 1j * math.sqrt(s.slice_s[l]) * (yl[:, l] @ dev["A"].reshape(case["G"], M * M))
        X = F[l + 1] @ _taylor(V.reshape(S, M, M), X.contiguous())
    return X


def _inputs(case, seed):
    """Everything a pass starts from; the same tensors for prepare() and exact()."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)
    s, dev = _system(case, gen)
    M, N, G, K, nw, P = (case[k] for k in ("M", "N", "G", "K", "nw", "P"))
    z = dict(generator=gen, device="cuda", dtype=F64)
    ctype = torch.complex64 if case["c64"] else C128
    spread = 0.3 / math.sqrt(M)
    pert = torch.complex(torch.randn(nw, 2, M, N, **z), torch.randn(nw, 2, M, N, **z))
    i = dict(phi=(dev["phi0"] + spread * pert).to(ctype))
    if case["ising"]:
        i["y"] = torch.where(torch.rand(nw, P, K, **z) < 0.5, -1.0, 1.0).to(F64)
    else:
        i["y"] = torch.randn(nw, P, K, **z)
    if case["kind"] != "trial":
        i["phiT"] = _trial(case, s, dev, i["y"].reshape(nw * P, K)).reshape(nw, P, M, N)
        i["logov"] = _logov(i["phi"], i["phiT"])
    if case["kind"] == "move":
        i["xi"] = torch.randn(nw, G, **z)
        i["xbar"] = 0.2 * torch.complex(torch.randn(nw, G, **z), torch.randn(nw, G, **z))
        i["eloc"] = torch.complex(-10.0 + torch.randn(nw, **z), 0.3 * torch.randn(nw, **z))
    if case["kind"] == "density":
        i["hist_xi"] = torch.randn(nw, max(case["h"], 1), G, **z)
        i["hist_xbar"] = 0.2 * torch.complex(torch.randn(nw, max(case["h"], 1), G, **z),
                                             torch.randn(nw, max(case["h"], 1), G, **z))
        i["w"] = 0.5 + torch.rand(nw, **z)
        i["phi_mid"] = i["phi"]
        i["phi_end"] = (dev["phi0"] + 1.2 * spread * pert.flip(0)).to(C128)
        i["logov"] = _logov(i["phi_end"], i["phiT"])
    return s, dev, i


def _overlap(phi, phiT):
    """Phi_T^T phi^s, [nw, P, 2, N, N]."""
    a = phiT.to(C128).transpose(-1, -2).contiguous()
    return torch.matmul(a[:, :, None], phi.to(C128)[:, None])


def _logov(phi, phiT):
    sign, logabs = torch.linalg.slogdet(_overlap(phi, phiT))
    return torch.complex(logabs.sum(-1), torch.angle(sign).sum(-1))


def _params(case, seed):
    p = ai.mlp_params(np.random.default_rng(seed), case["M"], case["K"], last_scale=0.05)
    p["b3"][case["K"]:] = 4 * np.arctanh(np.log(0.25) / 4)
    return p


def _context(case, s):
    kw = {}
    if case["learned"]:
        kw = dict(proposal=A.PROPOSAL_LEARNED, rw_step=0.5)
    elif not case["ising"]:
        kw = dict(proposal=A.PROPOSAL_RW, rw_step=0.08 if case["slices"] else 0.3)
    return A.Context(s, case["P"], _dtau(case), n_taylor=TAYLOR, weight_mode=A.WEIGHT_LOCAL,
                     max_walkers=case["nw"], xbar_cap=1.0, precision=case["prec"],
                     walker_c64=bool(case["c64"]), **kw)


class _State:
    pass


def prepare(case, seed):
    s, dev, i = _inputs(case, seed)
    st = _State()
    st.case, st.seed, st.i = case, int(seed), 0
    st.ctx = _context(case, s)
    if case["learned"]:
        A.afqmc_mlp_init(st.ctx, A.PREC_BF16, _params(case, seed), lr=1e-3)
        A.afqmc_mlp_set_training(st.ctx, True)
    st.w = D.Walkers(st.ctx, case["nw"])
    for name in ("phi", "y", "phiT", "logov", "xi", "xbar", "eloc"):
        if name in i:
            getattr(st.w, name).copy_(i[name])
    st.inp = i if case["kind"] in ("move", "paths", "density") else None
    nw, P, M, N = case["nw"], case["P"], case["M"], case["N"]
    if case["kind"] == "step":
        st.est = torch.zeros(2, dtype=F64, device="cuda")
    if case["kind"] in ("energy", "trial"):
        st.e_sample = torch.zeros(nw, P, dtype=C128, device="cuda")
    if case["kind"] == "paths":
        st.w.ref.copy_(torch.exp(1j * i["logov"].imag).sum(1))
    if case["kind"] == "density":
        z = dict(device="cuda", dtype=C128)
        st.bra = torch.zeros(nw, P, M, N, **z)
        st.theta = torch.zeros(nw, P, 2, M, N, **z)
        st.lbp = torch.zeros(nw, P, **z)
        st.rho = torch.zeros(nw, M, M, **z)
        st.out = torch.zeros(M * M + 1, dtype=F64, device="cuda")
    return st


def run(st):
    return _RUN[st.case["kind"]](st, st.case, st.ctx, st.w)


def _run_step(st, c, ctx, w):
    D.step(ctx, w, st.seed, st.i, st.est, n_sweep=c["sweeps"], n_qr=10, n_pc=1)
    st.i += 1
    return {"est": st.est, "phi": w.phi, "w": w.w, "y": w.y, "phiT": w.phiT, "logov": w.logov,
            "eloc": w.eloc, "xbar": w.xbar, "nacc": w.nacc}


def _run_energy(st, c, ctx, w):
    A.afqmc_green(ctx, w.nw, w.phi, w.phiT, w.logov, w.theta)
    A.afqmc_local_energy(ctx, w.nw, w.phiT, w.theta, w.logov, w.eloc, st.e_sample, w.xbar)
    return {"theta": w.theta, "logov": w.logov, "eloc": w.eloc, "e_sample": st.e_sample,
            "xbar": w.xbar}


def _run_trial(st, c, ctx, w):
    A.afqmc_trial_build(ctx, w.nw, w.y, w.phiT)
    return {"phiT": w.phiT, **_run_energy(st, c, ctx, w)}


def _run_move(st, c, ctx, w):
    # the pre-move walkers stay (a program that back-propagates keeps them)
    w.phi.copy_(st.inp["phi"])
    w.w.fill_(1.0)
    A.afqmc_propagate(ctx, w.nw, w.phi, w.xi, w.xbar, w.phiT, w.logov, -10.0, w.w, w.ref,
                      w.logov_new, w.eloc)
    A.afqmc_reorthogonalize(ctx, w.nw, w.phi, w.logov_new)
    return {"phi": w.phi, "w": w.w, "ref": w.ref, "logov_new": w.logov_new}


def _run_paths(st, c, ctx, w):
    w.w.fill_(1.0)
    A.afqmc_metropolis_x(ctx, w.nw, w.phi, w.y, w.phiT, w.logov, w.ref, w.w, st.seed, st.i,
                         c["sweeps"], w.nacc)
    st.i += 1
    return {"y": w.y, "phiT": w.phiT, "logov": w.logov, "w": w.w, "nacc": w.nacc}


def _run_density(st, c, ctx, w):
    i, h = st.inp, c["h"]
    A.afqmc_bp_density(ctx, w.nw, h, i["phi_mid"], i["hist_xi"] if h else None,
                       i["hist_xbar"] if h else None, w.phiT, w.logov, i["w"], st.bra, st.theta,
                       st.lbp, st.rho, st.out)
    return {"rho": st.rho, "out": st.out}


_RUN = {"step": _run_step, "energy": _run_energy, "trial": _run_trial, "move": _run_move,
        "paths": _run_paths, "density": _run_density}


# ---------------------------------------------------------------------------
# the same quantities in 64 bits


def _exact_energy(case, dev, phi, phiT):
    nw, P, M, N, G = (case[k] for k in ("nw", "P", "M", "N", "G"))
    S = nw * P
    theta = torch.matmul(phi.to(C128)[:, None], torch.linalg.inv(_overlap(phi, phiT)))
    S_p = torch.exp(1j * _logov(phi, phiT).imag)
    real = not phiT.is_complex()
    T = phiT.reshape(S, M, N)
    left = T.transpose(1, 2).reshape(S * N, M).contiguous()
    th = theta.reshape(S, 2, M, N)
    h1p = dev["h1"] + 0.5 * torch.matmul(dev["L"], dev["L"]).sum(0)
    cols = torch.cat([th[:, 0].real, th[:, 0].imag, th[:, 1].real, th[:, 1].imag], -1).contiguous()
    thc = torch.cat([th[:, 0], th[:, 1]], -1).contiguous()
    e = torch.zeros(S, dtype=C128, device="cuda")
    vb = torch.zeros(S, G, dtype=C128, device="cuda")
    for g in range(G + 1):
        Lg = dev["L"][g] if g < G else h1p
        if real:
            f = torch.bmm((left @ Lg).reshape(S, N, M), cols)
            f = [torch.complex(f[..., 2 * q * N:(2 * q + 1) * N], f[..., (2 * q + 1) * N:(2 * q + 2) * N])
                 for q in range(2)]
        else:
            f = torch.bmm((left @ Lg.to(C128)).reshape(S, N, M), thc)
            f = [f[..., :N], f[..., N:]]
        tr = sum(torch.diagonal(x, dim1=1, dim2=2).sum(-1) for x in f)
        if g < G:
            vb[:, g] = tr
            e += 0.5 * (tr * tr - sum((x * x.transpose(1, 2)).sum((1, 2)) for x in f))
        else:
            e += tr
    den = S_p.sum(1)
    eloc = (S_p * e.reshape(nw, P)).sum(1) / den
    xbar = -1j * math.sqrt(_dtau(case)) * (S_p[..., None] * vb.reshape(nw, P, G)).sum(1) / den[:, None]
    mag = xbar.abs()
    xbar = torch.where(mag > 1.0, xbar / mag, xbar)
    return {"theta": theta, "logov": None, "eloc": eloc, "e_sample": e.reshape(nw, P), "xbar": xbar}


def _field(case, dev, x):
    M = case["M"]
    b = dev["L"].reshape(case["G"], M * M)
    re, im = x.real.contiguous() @ b, x.imag.contiguous() @ b
    return (1j * math.sqrt(_dtau(case)) * torch.complex(re, im)).reshape(-1, M, M)


def _exact_move(case, dev, i):
    nw, M, N = case["nw"], case["M"], case["N"]
    Eh = dev["Eh"].to(C128)
    phi = i["phi"].to(C128).transpose(1, 2).reshape(nw, M, 2 * N)
    phi = Eh @ _taylor(_field(case, dev, i["xi"] - i["xbar"]), (Eh @ phi).contiguous())
    phi = phi.reshape(nw, M, 2, N).transpose(1, 2).contiguous()
    lnew, lold = _logov(phi, i["phiT"]), i["logov"]
    num = torch.exp(lnew - lold.real).sum(1)
    r = num / torch.exp(1j * lold.imag).sum(1)
    w = torch.exp(-_dtau(case) * (i["eloc"].real + 10.0)) * torch.clamp(torch.cos(torch.angle(r)), min=0.0)
    q, rr = torch.linalg.qr(phi)
    d = torch.diagonal(rr, dim1=-2, dim2=-1)
    return {"phi": q * (d / d.abs())[..., None, :], "w": w, "ref": num, "logov_new": None}


def _exact_density(case, dev, i):
    nw, P, M, N, h = (case[k] for k in ("nw", "P", "M", "N", "h"))
    Eh = dev["Eh"].to(C128)
    X = i["phiT"].to(C128).transpose(1, 2).reshape(nw, M, P * N)
    for t in range(h - 1, -1, -1):
        V = _field(case, dev, i["hist_xi"][:, t] - i["hist_xbar"][:, t])
        X = Eh @ _taylor(V, (Eh @ X).contiguous())
    bra = X.reshape(nw, M, P, N).transpose(1, 2).contiguous()
    lt = _logov(i["phi_mid"], bra)
    theta = torch.matmul(i["phi_mid"][:, None], torch.linalg.inv(_overlap(i["phi_mid"], bra)))
    la = lt - i["logov"].real
    a = torch.exp(la - la.real.max(1, keepdim=True).values)
    R = torch.matmul(theta.sum(2), bra.transpose(-1, -2).contiguous())
    R = (a[..., None, None] * R).sum(1) / a.sum(1)[:, None, None]
    out = torch.cat([(i["w"][:, None, None] * R.real).sum(0).reshape(-1), i["w"].sum().reshape(1)])
    return {"rho": R, "out": out}


def exact(case, seed):
    if case["kind"] in ("step", "paths"):  # many random accept tests: no closed value
        return None
    s, dev, i = _inputs(case, seed)
    if case["kind"] == "energy":
        return _exact_energy(case, dev, i["phi"], i["phiT"])
    if case["kind"] == "trial":
        nw, P, K = case["nw"], case["P"], case["K"]
        phiT = _trial(case, s, dev, i["y"].reshape(nw * P, K)).reshape(nw, P, case["M"], case["N"])
        return {"phiT": phiT, **_exact_energy(case, dev, i["phi"], phiT)}
    if case["kind"] == "move":
        return _exact_move(case, dev, i)
    return _exact_density(case, dev, i)


# ---------------------------------------------------------------------------
# what one pass cannot do without


def work(case):
    M, N, G, K, nw, P = (case[k] for k in ("M", "N", "G", "K", "nw", "P"))
    S, kind = nw * P, case["kind"]
    walker = nw * 2 * M * N * (8 if case["c64"] else 16)
    tcx = 2 if case["slices"] else 1                      # real or complex trial
    phiT = S * M * N * 8 * tcx
    L = (G + 1) * M * M * 8
    ov = S * 2 * (4 * tcx * M * N * N + 8 * N ** 3 / 3)    # overlap matrices and their LU
    green = ov + S * 2 * (16 * N ** 3 / 3 + 8 * M * N * N)
    if case["slices"]:
        contract = S * G * (4 * N * M * M + 2 * (8 * M * N * N + 8 * N * N))
    else:
        contract = S * G * (2 * N * M * M + 2 * (4 * M * N * N + 8 * N * N))
    move = nw * (4 * G * M * M + 2 * N * (TAYLOR * 8 + 8) * M * M)
    qr = nw * 2 * 8 * M * N * N
    if case["ising"]:
        trial, gens = S * (2 * K * M + M * N), K * M * 8
    elif case["slices"]:
        m = case["slices"]
        trial, gens = S * m * (2 * G * M * M + (TAYLOR + 1) * 4 * M * M * N), m * M * M * 8
    else:
        trial, gens = S * (2 * K * M * M + 20 * 2 * M * M * N), K * M * M * 8
    moves = case["sweeps"] * (K if case["ising"] else 1)
    nets = 0
    if case["learned"]:
        moves = 2 * case["sweeps"]
        H = A.MLP_HIDDEN
        one = 2 * S * ((M + K) * H + H * H + 2 * H * K)
        nets = case["sweeps"] * 5 * one               # three forward passes, one backward
    est = nw * G * 16 + S * 16 * 2
    if kind == "step":
        return {"bytes": 2 * walker + 2 * phiT + L + gens + est + 2 * S * K * 8,
                "flops": green + contract + move + ov + moves * (trial + ov)}
    if kind == "energy":
        return {"bytes": walker + phiT + L + S * 2 * M * N * 16 + est, "flops": green + contract}
    if kind == "trial":
        return {"bytes": walker + S * K * 8 + phiT + L + gens + S * 2 * M * N * 16 + est,
                "flops": trial + green + contract}
    if kind == "move":
        return {"bytes": 2 * walker + phiT + L + nw * G * 24 + S * 32, "flops": move + qr + ov}
    if kind == "paths":
        return {"bytes": walker + 2 * phiT + 2 * S * K * 8 + gens + S * 32,
                "flops": moves * (trial + ov) + nets}
    back = case["h"] * nw * (4 * G * M * M + P * N * (TAYLOR * 8 + 8) * M * M)
    return {"bytes": walker + phiT + L + nw * case["h"] * G * 24 + nw * M * M * 16 + M * M * 8,
            "flops": back + ov + S * (8 * M * N * N * 2 + 8 * M * M * N)}
