"""Performance cases of the library: what they run, on which inputs, how much
work that is, and what the results are in plain 64-bit torch.

A case is a dict of plain values.  `kind` names the call sequence:

  eval    one evaluation of every walker at new positions
  vmc     a run of Metropolis moves from the walkers' present state and the
          measurement after it (the step of a variational run)
  moves   a propose / accept loop in the caller's own program (drift wanted)
  grad    log|Psi| and E_loc through the autograd function, forward and backward
  logder  per-walker logarithmic derivatives of every parameter
  lrdmc   one iteration of lattice-regularised diffusion
  sr      one stochastic-reconfiguration solve
  multi   several systems of uneven size moved together, one graph replayed

A system is described by `atoms` (element symbols with counts), the electrons
per spin, the cube's side, the basis shells per atom (lower case Gaussian, upper
case Slater) with the range of their exponents, and options.  Everything else
is drawn from the seed.
"""
import math
import re
from types import SimpleNamespace

import numpy as np
import torch

import paper_2002_07401_amd as P

PRECISION = {"fp64": P.QMC_FP64, "refined": P.QMC_REFINED, "mixed": P.QMC_MIXED, "fp32": P.QMC_W_FP32,
             "bf16": P.QMC_MIXED_BF16}
CHARGE = {"H": 1, "He": 2, "Li": 3, "Be": 4, "B": 5, "C": 6, "N": 7, "O": 8}
N_COMP = {"s": 1, "p": 3, "d": 5}
L_OF = {"s": 0, "p": 1, "d": 2}
F64 = torch.float64

MOL160 = dict(atoms="H20 C10 O10", n_up=80, n_dn=80, box=20.0, shells="ssssppd", zmin=0.05, zmax=20.0,
              lam="lowrank", every=32)
MOL80 = dict(atoms="H10 C5 O5", n_up=40, n_dn=40, box=15.9, shells="ssssssppp", zmin=0.05, zmax=20.0,
             lam="gauss", j2=2, every=32)
ATOMS20 = dict(atoms="He1 Be1 C1 O1", n_up=10, n_dn=10, box=8.0, zmin=0.1, zmax=10.0, lam="gauss", every=32)


def listed():
    return [
        # the smallest call: a light molecule's few walkers evaluated once; launches and latency are all of it
        dict(name="eval_10e", kind="eval", atoms="He1 Li1 B1", n_up=5, n_dn=5, box=6.0, shells="sssssspp",
             axes=1, zmin=0.1, zmax=10.0, lam="gauss", every=32, precision="fp64", walkers=64),
        # a small open-shell molecule with unpaired orbitals and a three-body Jastrow: a short variational run
        dict(name="vmc_20e_open", kind="vmc", **{**ATOMS20, "n_up": 11, "n_dn": 9}, shells="ssspd", jshells="ssp",
             precision="fp64", walkers=256, moves=100),
        # the benchmark workload in both conforming precisions: one sweep of a 160-electron molecule and its measurement
        dict(name="vmc_160e", kind="vmc", **MOL160, precision="fp64", walkers=1024, moves=160),
        dict(name="vmc_160e_refined", kind="vmc", **MOL160, precision="refined", walkers=1024, moves=160),
        # a large system with a banded pairing matrix: part of a sweep and the measurement
        dict(name="vmc_1024e", kind="vmc", atoms="H32 He32 Li32 Be32 B32 C32 N32 O32", n_up=512, n_dn=512, box=40.0,
             shells="sssssppd", zmin=0.05, zmax=20.0, lam="band", every=64, precision="fp64", walkers=64, moves=64),
        # the Pfaffian pairing of an 80-electron molecule: one sweep and the measurement
        dict(name="vmc_80e_pfaffian", kind="vmc", **MOL80, pfaffian=1, precision="fp64", walkers=512, moves=80),
        # a caller's own move loop (its own acceptance rule, drift of the moved electron) over FP32 rows
        dict(name="moves_20e_mixed", kind="moves", **ATOMS20, shells="SSsPpD", precision="mixed", walkers=32),
        # forces on the nuclei and parameter gradients of an 80-electron molecule, forward and backward
        dict(name="grad_80e", kind="grad", **MOL80, precision="fp64", walkers=512),
        # the samples of an optimisation step of a small molecule: logarithmic derivatives, walker by walker
        dict(name="logder_20e", kind="logder", **ATOMS20, shells="ssspd", jshells="ssp", precision="fp64", walkers=1024),
        # diffusion: hop ratios, the continuous-time step and the next evaluation
        dict(name="lrdmc_160e", kind="lrdmc", **MOL160, precision="fp64", walkers=1024, a=0.1, a_valence=0.4, gamma=0.5,
             tau=0.05),
        # the optimiser's linear solve
        dict(name="sr_4096x8192", kind="sr", samples=4096, params=8192, eps=1e-3),
        # eight systems of 16 to 256 electrons as one group: 768 steps, the schedule period of all of them
        dict(name="multi_16_256e", kind="multi", sizes="16 32 48 64 96 128 192 256", precision="refined", walkers=256,
             moves=768, graph=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["eval", "eval", "vmc", "vmc", "vmc", "moves", "grad", "logder", "lrdmc", "sr", "multi"])
    if kind == "sr":
        return dict(kind=kind, samples=_log_int(rng, 48, 4096), params=_log_int(rng, 96, 8192),
                    eps=rng.choice([1e-3, 1e-2]))
    if kind == "multi":
        sizes = sorted(2 * _log_int(rng, 4, 100) for _ in range(rng.randint(2, 6)))
        return dict(kind=kind, sizes=" ".join(map(str, sizes)), precision=rng.choice(["refined", "fp64"]),
                    walkers=_log_int(rng, 16, 256), moves=_log_int(rng, 24, 192), graph=rng.randint(0, 1))
    small = kind in ("moves", "logder")
    n_at = _log_int(rng, 2, 8 if small else 40)
    names = [rng.choice(list(CHARGE)) for _ in range(n_at)]
    atoms = " ".join("%s%d" % (k, names.count(k)) for k in CHARGE if k in names)
    n = max(4, min(160, sum(CHARGE[k] for k in names)))
    c = dict(kind=kind, atoms=atoms, box=round(5.0 * n_at ** (1 / 3) + 1.0, 1), zmin=0.1, zmax=10.0, lam="gauss",
             every=rng.choice([16, 32, 64]), j2=rng.randint(1, 2), precision="fp64")
    extra = rng.choice([0, 0, 1, 2]) if kind != "grad" else 0
    c["n_dn"] = (n - extra) // 2
    c["n_up"] = n - c["n_dn"]
    if c["n_up"] - c["n_dn"] > 2 or kind == "grad":
        c["n_up"] = c["n_dn"]
    # enough functions for a regular geminal matrix, and an uneven number of them
    per = max(rng.randint(5, 15), -(-2 * c["n_up"] // n_at))
    shells, have = "", 0
    for s in ["s", "s", "p", "s", "d", "p", "s", "p", "d", "s"] * 40:
        if have >= per:
            break
        shells, have = shells + s, have + N_COMP[s]
    c["shells"] = shells
    c["lam"] = "gauss"
    if kind in ("eval", "vmc"):
        c["precision"] = rng.choice(["fp64", "fp64", "refined"])
        opt = rng.choice(["", "", "pfaffian", "jastrow", "slater", "contract"])
        if opt == "pfaffian" and n <= 92 and n % 2 == 0:
            c.update(pfaffian=1, n_up=n - c["n_dn"], unpaired=2 if extra else 0)
        elif opt == "jastrow":
            c.update(jshells="ssp", precision="fp64")
        elif opt == "slater":
            c["shells"] = c["shells"].replace("p", "P", 1).replace("s", "S", 1)
        elif opt == "contract":
            c.update(contract=max(4, -(-2 * c["n_up"] // n_at) * 2 // 3), precision="fp64")
    if kind == "moves":
        c["precision"] = rng.choice(["fp64", "mixed", "fp32", "refined"])
    if kind == "logder":
        c["jshells"] = rng.choice(["", "ssp"])
    if kind == "lrdmc":
        c.update(a=0.1, a_valence=rng.choice([0.0, 0.4]), gamma=rng.choice([0.0, 0.5]), tau=0.05)
    c["walkers"] = _log_int(rng, 16, {"grad": 512, "logder": 512, "moves": 512}.get(kind, 1024))
    if kind == "vmc":
        c["moves"] = c["n_up"] + c["n_dn"]
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _functions(rng, n_at, spec, lo, hi, axes=False):
    """Basis functions of every atom: centre, l, m, radial, zeta (one exponent a shell).
    axes: a "p" is a single component, its axis cycling over the system."""
    c, l, m, rad, z = [], [], [], [], []
    axis = 0
    for a in range(n_at):
        for s in spec:
            slater = s.isupper()
            zeta = math.exp(rng.uniform(math.log(0.5 if slater else lo), math.log(5.0 if slater else hi)))
            ll = L_OF[s.lower()]
            comps = range(N_COMP[s.lower()])
            if axes and ll == 1:
                comps, axis = [axis % 3], axis + 1
            for mm in comps:
                c.append(a), l.append(ll), m.append(mm), rad.append(int(slater)), z.append(zeta)
    i32 = lambda v: np.array(v, np.int32)  # noqa: E731
    return i32(c), i32(l), i32(m), i32(rad), np.array(z)


def _sym(rng, n, scale):
    a = np.triu(rng.standard_normal((n, n)) * scale)
    return a + np.triu(a, 1).T


def _skew(rng, n, scale):
    a = np.triu(rng.standard_normal((n, n)) * scale, 1)
    return a - a.T


def _system(case, rng):
    """The molecule as JAGPSystem takes it."""
    Z = np.concatenate([np.full(int(k), float(CHARGE[e])) for e, k in re.findall(r"([A-Z][a-z]?)(\d+)", case["atoms"])])
    A = len(Z)
    R = np.empty((0, 3))
    while len(R) < A:
        p = rng.uniform(0.0, case["box"], 3)
        if not len(R) or np.min(np.linalg.norm(R - p, axis=1)) >= 1.0:
            R = np.vstack([R, p])
    center, l, m, radial, zeta = _functions(rng, A, case["shells"], case["zmin"], case["zmax"], bool(case.get("axes")))
    n_prim = len(zeta)
    C = None
    if case.get("contract"):
        k = case["contract"]
        C = np.zeros((n_prim, A * k))
        for a in range(A):
            own = np.nonzero(center == a)[0]
            C[np.ix_(own, np.arange(a * k, (a + 1) * k))] = rng.standard_normal((len(own), k)) / 4.0
    L = n_prim if C is None else C.shape[1]
    if case["lam"] == "lowrank":
        f = rng.standard_normal((L, case["n_up"])) / math.sqrt(L)
        lam = f @ f.T + 1e-3 * _sym(rng, L, 1.0)
    elif case["lam"] == "band":
        near = (np.linalg.norm(R[:, None] - R[None], axis=-1) < 8.0)[center][:, center]
        lam = _sym(rng, L, 1.0 / math.sqrt(near.sum(1).mean())) * near
    else:
        lam = _sym(rng, L, 1.0 / L)
    k_open = case["n_up"] - case["n_dn"]
    j2 = np.array([1.0, 1.0]) if case.get("j2", 1) == 1 else np.array([1.0, 0.05, -0.02, 0.01, 1.0, 0.08, -0.03, 0.01])
    s = SimpleNamespace(R=R, Z=Z, center=center, l=l, m=m, radial=radial, zeta=zeta, lam=lam, n_up=case["n_up"],
                        n_dn=case["n_dn"], unpaired=rng.standard_normal((L, k_open)) / math.sqrt(L), j1_form=2,
                        j1_b=np.ones(A), j2_form=case.get("j2", 1), j2=j2, refresh_every=case["every"], contraction=C,
                        jb_zeta=None, pairing=0)
    if case.get("pfaffian"):
        k = case.get("unpaired", 0)
        s.pairing = 1
        s.lam = lam + _skew(rng, L, 0.3 / L)
        s.pf_uu, s.pf_dd = _skew(rng, L, 0.5 / L), _skew(rng, L, 0.5 / L)
        s.unpaired, s.unpaired_dn = (rng.standard_normal((L, k)) / math.sqrt(L) for _ in range(2))
    if case.get("jshells"):
        s.jb_center, s.jb_l, s.jb_m, s.jb_radial, s.jb_zeta = _functions(rng, A, case["jshells"], 0.2, 3.0)
        LJ = len(s.jb_zeta)
        s.j1_inh = 0.1 * rng.standard_normal((2, LJ))
        s.j3 = np.stack([_sym(rng, LJ, 0.05), _sym(rng, LJ, 0.05), 0.05 * rng.standard_normal((LJ, LJ))])
    return s


def _positions(s, rng, walkers):
    """Electrons around the nuclei in proportion to their charges, unit spread, spins alternating."""
    N = s.n_up + s.n_dn
    share = s.Z / s.Z.sum() * N
    count = np.floor(share).astype(int)
    count[np.argsort(-(share - count), kind="stable")[:N - count.sum()]] += 1
    owner = np.repeat(np.arange(len(s.Z)), count)
    lo = 2 * min(s.n_up, s.n_dn)
    up, dn = list(owner[0:lo:2]), list(owner[1:lo:2])
    (up if s.n_up >= s.n_dn else dn).extend(owner[lo:])
    return s.R[up + dn][None] + rng.standard_normal((walkers, N, 3))


def _member(n):
    """One helium-like system of n electrons of an uneven group."""
    return dict(atoms="He%d" % (n // 2), n_up=n // 2, n_dn=n // 2, box=(100.0 * n) ** (1 / 3), shells="sssssp", zmin=0.1,
                zmax=10.0, lam="gauss", every=32)


def _host_inputs(case, seed):
    """Everything a pass is made of, on the host, from the seed alone."""
    rng = np.random.default_rng(seed)
    x = SimpleNamespace()
    if case["kind"] == "multi":
        x.systems = [_system(_member(int(n)), rng) for n in case["sizes"].split()]
        x.r0 = [_positions(s, rng, case["walkers"]) for s in x.systems]
        x.key = int(rng.integers(1 << 40))
        return x
    x.s = _system(case, rng)
    N, Wk = case["n_up"] + case["n_dn"], case["walkers"]
    x.r0 = _positions(x.s, rng, Wk)
    if case["kind"] in ("vmc", "moves"):
        steps = case.get("moves", N)
        x.disp = 0.3 * rng.standard_normal((steps, Wk, 3))
        x.unif = rng.random((steps, Wk))
    if case["kind"] == "lrdmc":
        x.xi = rng.random((Wk, 2))
    if case["kind"] == "grad":
        x.gl, x.ge = rng.standard_normal((2, Wk)) / Wk
    return x


def _sr_inputs(case, seed):
    """Correlated logarithmic derivatives whose scales span two decades, and energies that depend on them."""
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(int(seed))
    M, K = case["samples"], case["params"]
    n0 = -(-K // 16)
    base = torch.randn(M, n0, generator=g, device=dev, dtype=F64)
    O = torch.randn(M, K, generator=g, device=dev, dtype=F64)
    O += base.repeat(1, 16)[:, :K]
    O *= torch.logspace(-1, 1, K, device=dev, dtype=F64)
    e = -5.0 + torch.randn(M, generator=g, device=dev, dtype=F64) + 0.5 * O[:, 0]
    return O, e


def prepare(case, seed):
    dev = torch.device("cuda:0")
    kind = case["kind"]
    t = lambda a: torch.tensor(a, device=dev)  # noqa: E731
    st = SimpleNamespace(case=case)
    if kind == "sr":
        st.O, st.e = _sr_inputs(case, seed)
        n = P.load().qmc_sr_workspace_size(case["samples"], case["params"])
        st.work = torch.empty((n + 7) // 8, dtype=F64, device=dev)
        return st
    x = _host_inputs(case, seed)
    prec = PRECISION[case["precision"]]
    if kind == "multi":
        st.walkers = [P.Walkers(P.JAGPSystem(s, precision=prec), case["walkers"], adjoint=False) for s in x.systems]
        for w, r0 in zip(st.walkers, x.r0):
            w.eval_batch(t(r0))
        st.group = P.MultiSystem(st.walkers)
        st.group.autotune()
        st.key = x.key
        return st
    st.sys = P.JAGPSystem(x.s, precision=prec)
    st.wk = P.Walkers(st.sys, case["walkers"], adjoint=kind in ("grad", "logder"))
    st.r = t(x.r0)
    if kind in ("vmc", "moves", "lrdmc"):
        st.wk.eval_batch(st.r)
    if kind in ("vmc", "moves"):
        st.disp, st.unif = t(x.disp), t(x.unif)
        st.count = torch.zeros(case["walkers"], dtype=torch.int32, device=dev)
        st.at = 0
    if kind == "moves":
        st.status = torch.zeros(case["walkers"], dtype=torch.int32, device=dev)
    if kind == "lrdmc":
        st.xi = t(x.xi)
        st.weight = torch.ones(case["walkers"], dtype=F64, device=dev)
        st.left = torch.full((case["walkers"],), case["tau"], dtype=F64, device=dev)
    if kind == "grad":
        st.gl, st.ge = t(x.gl), t(x.ge)
        s = x.s
        st.leaves = [st.r] + [t(np.ascontiguousarray(v)) for v in (s.R, s.zeta, s.lam, np.concatenate([s.j1_b, s.j2]))]
        for v in st.leaves:
            v.requires_grad_(True)
    if kind == "logder":
        st.ones = torch.ones(case["walkers"], dtype=F64, device=dev)
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(st):
    case = st.case
    kind = case["kind"]
    if kind == "eval":
        return st.wk.eval_batch(st.r)
    if kind == "vmc":
        st.wk.vmc_steps(st.at, st.disp, st.unif, st.count)
        st.at = (st.at + case["moves"]) % (case["n_up"] + case["n_dn"])
        out = st.wk.eval_batch(None)
        out["r"], out["count"] = st.wk.read(P.STATE_R), st.count
        return out
    if kind == "moves":
        ratios, drifts = [], []
        for e in range(case["n_up"] + case["n_dn"]):
            new = st.r[:, e] + st.disp[e]
            q, d = st.wk.propose(e, new, drift=True)
            ok = st.unif[e] < q * q
            st.wk.accept(e, ok.to(torch.uint8), st.status)
            st.r[:, e] = torch.where(ok.unsqueeze(1), new, st.r[:, e])
            ratios.append(q)
            drifts.append(d)
        return dict(ratios=torch.stack(ratios), drifts=torch.stack(drifts), r=st.r.clone(),
                    logabs=st.wk.read(P.STATE_LOGABS), status=st.status)
    if kind == "grad":
        for v in st.leaves:
            v.grad = None
        logabs, e_loc = P.JAGPFunction.apply(st.wk, *st.leaves)
        torch.autograd.backward([logabs, e_loc], [st.gl, st.ge])
        return dict(logabs=logabs.detach(), e_loc=e_loc.detach(), **{k: v.grad for k, v in
                    zip(("r", "R", "zeta", "lam", "jas"), st.leaves)})
    if kind == "logder":
        return st.wk.forces(st.r, st.ones, None, per_walker=True)
    if kind == "lrdmc":
        st.weight.fill_(1.0)
        st.left.fill_(case["tau"])
        g = st.wk.lrdmc_hops(case["a"], case["a_valence"], 1.0, case["gamma"])
        st.r, hop = st.wk.lrdmc_advance(st.xi, st.weight, st.left)
        out = st.wk.eval_batch(st.r, drift=False)
        return dict(ratios=g["ratios"], terms=g["terms"], r=st.r, hop=hop, weight=st.weight, left=st.left,
                    logabs=out["logabs"], sign=out["sign"], e_kin=out["e_kin"], e_loc=out["e_loc"],
                    status=out["status"])
    if kind == "sr":
        delta, f, _ = P.sr_step(st.O, st.e, case["eps"], work=st.work)
        return dict(delta=delta, force=f)
    st.group.vmc_steps(case["moves"], seed=st.key, sigma=0.3, use_graph=bool(case["graph"]))
    return {"%02d" % i: dict(r=w.read(P.STATE_R), logabs=w.read(P.STATE_LOGABS), sign=w.read(P.STATE_SIGN))
            for i, w in enumerate(st.walkers)}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _sizes(case):
    A = sum(int(k) for k in re.findall(r"[A-Z][a-z]?(\d+)", case["atoms"]))
    n_p = case["shells"].lower().count("p")
    per = sum(N_COMP[s.lower()] for s in case["shells"]) - (2 * n_p if case.get("axes") else 0)
    L = A * case["contract"] if case.get("contract") else A * per
    return A, L, case["n_up"], case["n_dn"]


def _eval_work(case):
    """Operations of one walker's evaluation: basis values and derivatives, the pairing products, the inverse,
    the cofactor products and the pair sums.  A banded pairing matrix counts by its share of nonzeros."""
    A, L, nu, nd = _sizes(case)
    N = nu + nd
    fill = min(1.0, (4.0 / 3.0) * math.pi * 8.0 ** 3 / case["box"] ** 3) if case["lam"] == "band" else 1.0
    if case.get("pfaffian"):
        n = N + case.get("unpaired", 0)
        det = 2 * (2 * N) * L * L + n * n * L + n ** 3 + 2 * n * n * L
    else:
        det = 2 * N * L * L * fill + 2 * nu * nu * L + 2 * nu ** 3 + 4 * nu * nu * L
    return 40.0 * N * A * max(1, L // A) + det + 40.0 * N * (N + A)


def _move_work(case):
    """Operations of one walker's move: basis values, the new row, the update of the inverse, the Jastrow change."""
    A, L, nu, nd = _sizes(case)
    N = nu + nd
    n = N if case.get("pfaffian") else nu
    return 20.0 * L + 2 * n * L * (2 if case.get("pfaffian") else 1) + 4.0 * n * n + 20.0 * (N + A)


def work(case):
    kind = case["kind"]
    if kind == "sr":
        M, K = case["samples"], case["params"]
        return {"bytes": 8.0 * M * K + 8.0 * M + 16.0 * K, "flops": 4.0 * M * K * 40}
    if kind == "multi":
        b = f = 0.0
        for n in map(int, case["sizes"].split()):
            c = _member(n)
            L = 4 * n
            b += case["walkers"] * (2 * 24.0 * n + 16.0) + 8.0 * L * L
            # every sweep's moves, and the pairing product of each spin once a sweep
            f += case["walkers"] * case["moves"] * (_move_work(c) + 2.0 * L * L)
        return {"bytes": b, "flops": f}
    A, L, nu, nd = _sizes(case)
    N, Wk = nu + nd, case["walkers"]
    io = Wk * (24.0 * N + 36.0) + 8.0 * L * L
    ev = Wk * _eval_work(case)
    if kind == "eval":
        return {"bytes": io + 24.0 * Wk * N, "flops": ev}
    if kind == "vmc":
        # the evaluation's pairing product is also what the moves read, so it is counted once
        return {"bytes": io + Wk * (32.0 * case["moves"] + 48.0 * N), "flops": ev + Wk * case["moves"] * _move_work(case)}
    if kind == "moves":
        return {"bytes": io + Wk * N * (24.0 + 8.0 + 32.0), "flops": Wk * N * _move_work(case)}
    if kind == "grad":
        return {"bytes": io + 24.0 * Wk * N + 8.0 * L * L, "flops": 4.0 * ev}
    if kind == "logder":
        LJ = A * sum(N_COMP[s] for s in case.get("jshells", ""))
        per = L * L + 2 * L + 3 * A + A + 3 * N + 3 * LJ * LJ + 3 * LJ
        return {"bytes": io + 8.0 * Wk * per, "flops": 2.0 * ev + 2.0 * Wk * (N / 2 * L * L + 3 * N * LJ * LJ)}
    hops = Wk * 6.0 * N
    return {"bytes": io + 8.0 * hops, "flops": ev + hops * (20.0 * L + 20.0 * (N + A))}


# ---------------------------------------------------------------------------
# the same results in plain 64-bit torch
# ---------------------------------------------------------------------------

class _Exact:
    """A system's wave function as its definition says, batched over walkers.  Parameters are tensors, and may be
    one set for all walkers or one for each (leading dimension)."""

    def __init__(self, s, dev):
        t = lambda a: torch.tensor(np.ascontiguousarray(a, dtype=np.float64), device=dev)  # noqa: E731
        i = lambda a: torch.tensor(np.asarray(a, dtype=np.int64), device=dev)  # noqa: E731
        self.s, self.dev, self.nu, self.N = s, dev, s.n_up, s.n_up + s.n_dn
        self.R, self.Z, self.zeta, self.lam, self.jas = t(s.R), t(s.Z), t(s.zeta), t(s.lam), t(np.concatenate([s.j1_b, s.j2]))
        self.kind = (i(s.center), i(s.l), i(s.m), i(s.radial))
        self.C = None if s.contraction is None else t(s.contraction)
        L = len(s.lam)
        self.U = t(np.asarray(s.unpaired).reshape(L, -1))
        if s.pairing:
            self.Uu, self.Ud = self.U, t(np.asarray(s.unpaired_dn).reshape(L, -1))
            self.uu, self.dd = t(s.pf_uu), t(s.pf_dd)
        self.LJ = 0 if s.jb_zeta is None else len(s.jb_zeta)
        if self.LJ:
            self.jkind = (i(s.jb_center), i(s.jb_l), i(s.jb_m), i(s.jb_radial))
            self.jzeta, self.j1, self.j3 = t(s.jb_zeta), t(s.j1_inh), t(s.j3)

    # -- basis ------------------------------------------------------------
    def _basis(self, r, kind, zeta, deriv):
        """Values [.., n, L] (and gradients [.., n, 3, L], Laplacians) at r [.., n, 3]; zeta [L] or [Wk, L]."""
        c, l, m, rad = kind
        R = self.R if self.R.dim() == 2 else self.R.unsqueeze(-3)
        d = r.unsqueeze(-2) - R                                      # [.., n, A, 3]
        x, y, z = d.unbind(-1)
        one, zero = torch.ones_like(x), torch.zeros_like(x)
        at = c * 9 + torch.where(l == 0, 0, torch.where(l == 1, 1, 4)) + m
        pick = lambda v: torch.stack(v, -1).flatten(-2).index_select(-1, at)  # noqa: E731
        Pm = pick([one, x, y, z, x * y, y * z, z * x, x * x - y * y, 2 * z * z - x * x - y * y])
        r2 = (d * d).sum(-1).index_select(-1, c)
        zt = zeta if zeta.dim() == 1 else zeta.unsqueeze(-2)
        gauss = rad == 0
        rr = torch.sqrt(torch.where(gauss, torch.ones_like(r2), r2))
        e = torch.exp(-zt * torch.where(gauss, r2, rr))
        psi = Pm * e
        if not deriv:
            return (psi,) if self.C is None or kind is not self.kind else (psi @ self.C,)
        over = torch.where(gauss, -2.0 * zt, -zt / rr)               # e' / (r e)
        ll = l.to(F64)
        lap = psi * torch.where(gauss, 4.0 * zt * zt * r2 - 2.0 * zt * (2.0 * ll + 3.0), zt * zt - 2.0 * zt * (ll + 1.0) / rr)
        gP = [pick([zero, one, zero, zero, y, zero, z, 2 * x, -2 * x]),
              pick([zero, zero, one, zero, x, z, zero, -2 * y, -2 * y]),
              pick([zero, zero, zero, one, zero, y, x, zero, 4 * z])]
        g = [e * (gP[k] + Pm * over * d[..., k].index_select(-1, c)) for k in range(3)]
        if self.C is not None and kind is self.kind:
            psi, lap, g = psi @ self.C, lap @ self.C, [v @ self.C for v in g]
        return psi, g, lap

    # -- Jastrow ------------------------------------------------------------
    def _radial(self, d2, same):
        """v(r), v'(r)/r and v'' + 2 v'/r of pairs at squared distance d2."""
        A = len(self.s.Z)
        j = self.jas[..., A:] if self.jas.dim() == 1 else self.jas[:, None, None, A:]
        h = j.shape[-1] // 2
        pr = [torch.where(same, j[..., k], j[..., h + k]) for k in range(h)]
        r = torch.sqrt(d2)
        c = torch.where(same, 0.25, 0.5).to(F64)
        a = pr[1:] if h == 4 else []
        q = 1.0 + pr[0] * r
        t = r / q
        v, v1, v2 = c * t, c, torch.zeros_like(r)
        for k, ak in enumerate(a):
            v, v1, v2 = v + ak * t ** (k + 2), v1 + (k + 2) * ak * t ** (k + 1), v2 + (k + 2) * (k + 1) * ak * t ** k
        t1, t2 = 1.0 / (q * q), -2.0 * pr[0] / q ** 3
        f1, f2 = v1 * t1, v2 * t1 * t1 + v1 * t2
        return v, f1 / r, f2 + 2.0 * f1 / r

    def _one_body(self, d2):
        A = len(self.s.Z)
        b = self.jas[:A] if self.jas.dim() == 1 else self.jas[:, None, :A]
        z2 = 2.0 * self.Z
        r = torch.sqrt(d2)
        q = 1.0 + b * z2 ** 0.25 * r
        f = -(z2 ** 0.75) * z2 ** 0.25 * r / (2.0 * q)
        f1 = -z2 * 0.5 / (q * q)
        f2 = z2 ** 1.25 * b / q ** 3
        return f, f1 / r, f2 + 2.0 * f1 / r

    def _up(self, n=None):
        return torch.arange(self.N, device=self.dev) < self.nu

    def jastrow(self, r):
        """J [Wk], its gradients [Wk, N, 3], Laplacians [Wk, N], and the Coulomb energy [Wk]."""
        R = self.R if self.R.dim() == 2 else self.R.unsqueeze(-3)
        d = r.unsqueeze(2) - R
        d2 = (d * d).sum(-1)
        f, g1, l1 = self._one_body(d2)
        J, g, h = f.sum((1, 2)), (g1.unsqueeze(-1) * d).sum(2), l1.sum(2)
        V = -(self.Z / torch.sqrt(d2)).sum((1, 2))
        eye = torch.eye(self.N, device=self.dev, dtype=F64)
        d = r.unsqueeze(2) - r.unsqueeze(1)
        d2 = (d * d).sum(-1) + eye
        up = self._up()
        v, g1, l1 = self._radial(d2, up.unsqueeze(0) == up.unsqueeze(1))
        off = 1.0 - eye
        J, g, h = J + 0.5 * (v * off).sum((1, 2)), g + ((g1 * off).unsqueeze(-1) * d).sum(2), h + (l1 * off).sum(2)
        V = V + 0.5 * (off / torch.sqrt(d2)).sum((1, 2))
        if len(self.s.Z) > 1:
            ia = torch.triu_indices(len(self.s.Z), len(self.s.Z), 1, device=self.dev)
            dn = self.R[..., ia[0], :] - self.R[..., ia[1], :]
            V = V + (self.Z[ia[0]] * self.Z[ia[1]] / torch.sqrt((dn * dn).sum(-1))).sum(-1)
        if self.LJ:
            chi, gc, lc = self._basis(r, self.jkind, self.jzeta, True)
            field = self._field(chi)
            own = torch.cat([chi[:, :self.nu] @ self.j3[..., 0, :, :], chi[:, self.nu:] @ self.j3[..., 1, :, :]], 1)
            j1 = self.j1 if self.j1.dim() == 3 else self.j1.unsqueeze(0)
            lin = torch.cat([j1[:, :1].expand(-1, self.nu, -1), j1[:, 1:].expand(-1, self.N - self.nu, -1)], 1)
            pair = field - own                                       # sum over the other electrons
            J = J + (lin * chi).sum((1, 2)) + 0.5 * (pair * chi).sum((1, 2))
            g = g + torch.stack([((lin + pair) * v).sum(-1) for v in gc], -1)
            h = h + ((lin + pair) * lc).sum(-1)
        return J, g, h, V

    def _field(self, chi):
        """sum_j M^{s_i s_j} chi(r_j) over all electrons j, for every i."""
        X = torch.stack([chi[:, :self.nu].sum(1), chi[:, self.nu:].sum(1)], 1)
        M = self.j3
        fu = (M[..., 0, :, :] @ X[:, 0, :, None] + M[..., 2, :, :] @ X[:, 1, :, None]).squeeze(-1)
        fd = (M[..., 1, :, :] @ X[:, 1, :, None] + M[..., 2, :, :].transpose(-1, -2) @ X[:, 0, :, None]).squeeze(-1)
        return torch.cat([fu.unsqueeze(1).expand(-1, self.nu, -1), fd.unsqueeze(1).expand(-1, self.N - self.nu, -1)], 1)

    # -- pairing ------------------------------------------------------------
    def rows(self, psi):
        """Q [Wk, N, n, L] is never formed; this gives P with W = P_up psi_dn^T: psi_up Lambda and psi_dn Lambda^T."""
        return torch.cat([psi[:, :self.nu] @ self.lam, psi[:, self.nu:] @ self.lam.transpose(-1, -2)], 1)

    def matrix(self, psi):
        """The geminal matrix, or the pairing matrix of the Pfaffian with its fictitious rows."""
        u, d = psi[:, :self.nu], psi[:, self.nu:]
        if not self.s.pairing:
            return torch.cat([u @ self.lam @ d.transpose(1, 2), u @ self.U], 2)
        ud = u @ self.lam @ d.transpose(1, 2)
        G = torch.cat([torch.cat([u @ self.uu @ u.transpose(1, 2), ud], 2),
                       torch.cat([-ud.transpose(1, 2), d @ self.dd @ d.transpose(1, 2)], 2)], 1)
        F = torch.cat([u @ self.Uu, d @ self.Ud], 1)
        k = F.shape[2]
        zero = torch.zeros(len(G), k, k, dtype=F64, device=self.dev)
        G = torch.cat([torch.cat([G, F], 2), torch.cat([-F.transpose(1, 2), zero], 2)], 1)
        return 0.5 * (G - G.transpose(1, 2))

    def logdet(self, W):
        """log|.| and sign of the determinant, or of the Pfaffian (Parlett-Reid with exchanges)."""
        if not self.s.pairing:
            sign, la = torch.linalg.slogdet(W)
            return la, sign
        A, n = W.clone(), W.shape[1]
        b = torch.arange(len(A), device=self.dev)
        la, sign = torch.zeros(len(A), dtype=F64, device=self.dev), torch.ones(len(A), dtype=F64, device=self.dev)
        for k in range(0, n - 1, 2):
            p = k + 1 + A[:, k, k + 1:].abs().argmax(1)
            sign = torch.where(p == k + 1, sign, -sign)
            perm = torch.arange(n, device=self.dev).repeat(len(A), 1)
            perm[b, p] = k + 1
            perm[:, k + 1] = p
            A = A.gather(1, perm.unsqueeze(2).expand(-1, -1, n)).gather(2, perm.unsqueeze(1).expand(-1, n, -1))
            a = A[:, k, k + 1]
            la, sign = la + a.abs().log(), sign * a.sign()
            tau, row = A[:, k, k + 2:] / a.unsqueeze(1), A[:, k + 1, k + 2:].clone()
            A[:, k + 2:, k + 2:] += row.unsqueeze(2) * tau.unsqueeze(1) - tau.unsqueeze(2) * row.unsqueeze(1)
        return la, sign

    def cofactors(self, psi, inv):
        """Y [Wk, N, L] with the determinant's (Pfaffian's) derivative along psi(r_i) being Y_i."""
        u, d = psi[:, :self.nu], psi[:, self.nu:]
        if not self.s.pairing:
            nd = self.N - self.nu
            yu = inv[:, :nd].transpose(1, 2) @ d @ self.lam.transpose(-1, -2)
            if self.U.shape[-1]:
                yu = yu + inv[:, nd:].transpose(1, 2) @ self.U.transpose(-1, -2)
            return torch.cat([yu, inv[:, :nd] @ u @ self.lam], 1)
        G = inv[:, :self.N, :self.N].transpose(1, 2)                 # G[i, j] = inv[j, i]
        yu = G[:, :self.nu, :self.nu] @ u @ self.uu.T + G[:, :self.nu, self.nu:] @ d @ self.lam.T
        yd = -(G[:, self.nu:, :self.nu] @ u @ self.lam) + G[:, self.nu:, self.nu:] @ d @ self.dd.T
        y = torch.cat([yu, yd], 1)
        k = self.Uu.shape[1]
        if k:
            F = inv[:, self.N:, :self.N].transpose(1, 2)
            y = y + torch.cat([F[:, :self.nu] @ self.Uu.T, F[:, self.nu:] @ self.Ud.T], 1)
        return y

    def evaluate(self, r):
        psi, g, lap = self._basis(r, self.kind, self.zeta, True)
        W = self.matrix(psi)
        la, sign = self.logdet(W)
        y = self.cofactors(psi, torch.linalg.inv(W))
        D = torch.stack([(v * y).sum(-1) for v in g], -1)
        J, gJ, hJ, V = self.jastrow(r)
        e_kin = -0.5 * ((lap * y).sum(-1) + 2.0 * (D * gJ).sum(-1) + hJ + (gJ * gJ).sum(-1)).sum(-1)
        return dict(logabs=la + J, sign=sign, drift=D + gJ, e_kin=e_kin, e_loc=e_kin + V, y=y)

    def in_parts(self, r, walkers_at_once):
        parts = [self.evaluate(p) for p in r.split(walkers_at_once)]
        return {k: torch.cat([p[k] for p in parts]) for k in parts[0]}

    # -- moves --------------------------------------------------------------
    def d_jastrow(self, r, e, x, chi=None):
        """Change of J when electrons e go to x [Wk, 3] (and its gradient there)."""
        up = self._up()
        others = torch.arange(self.N, device=self.dev) != e
        J, g = [], None
        for p in (r[:, e], x):
            d = p.unsqueeze(1) - self.R
            f, g1, _ = self._one_body((d * d).sum(-1))
            j, g = f.sum(1), (g1.unsqueeze(-1) * d).sum(1)
            d = (p.unsqueeze(1) - r)[:, others]
            v, g1, _ = self._radial((d * d).sum(-1), (up == up[e])[others])
            J.append(j + v.sum(1))
            g = g + (g1.unsqueeze(-1) * d).sum(1)
        dJ = J[1] - J[0]
        if self.LJ:
            s = 0 if e < self.nu else 1
            new, gc, _ = self._basis(x.unsqueeze(1), self.jkind, self.jzeta, True)
            new = new.squeeze(1)
            lin = self.j1[s] + (self._field(chi)[:, e] - chi[:, e] @ self.j3[s])
            dJ = dJ + ((new - chi[:, e]) * lin).sum(1)
            g = g + torch.stack([(v.squeeze(1) * lin).sum(-1) for v in gc], -1)
            chi = chi.clone()
            chi[:, e] = new
        return dJ, g, chi

    def chain(self, r, disp, unif, drift=False):
        """Metropolis moves of electron t mod N; the ratios, drifts and how many were accepted besides."""
        r = r.clone()
        psi = self._basis(r, self.kind, self.zeta, False)[0]
        chi = self._basis(r, self.jkind, self.jzeta, False)[0] if self.LJ else None
        ratios, drifts, count = [], [], torch.zeros(len(r), dtype=torch.int32, device=self.dev)
        pf, spin, inv = bool(self.s.pairing), -1, None
        nd = self.N - self.nu
        for t in range(len(disp)):
            e = t % self.N
            s = 0 if e < self.nu else 1
            if pf or s != spin or t % 16 == 0:                       # afresh; between, rank-one updates
                W = self.matrix(psi)
                inv = torch.linalg.inv(W)
                # the fixed vectors that psi(r') of this spin is paired with
                if not pf:
                    fixed = psi[:, self.nu:] @ self.lam.T if s == 0 else psi[:, :self.nu] @ self.lam
                    if s == 0 and self.U.shape[1]:
                        fixed = torch.cat([fixed, self.U.T.expand(len(r), -1, -1)], 1)
                spin = s
            x = r[:, e] + disp[t]
            out = self._basis(x.unsqueeze(1), self.kind, self.zeta, drift)
            new = out[0].squeeze(1)
            if pf:
                y = self.cofactors(psi, inv)[:, e]
                ratio = (new * y).sum(1)
            else:
                row = (fixed @ new.unsqueeze(2)).squeeze(2)          # the new row (up) or column (down)
                col = inv[:, :, e] if s == 0 else inv[:, e - self.nu]
                ratio = (row * col).sum(1)
                y = (col.unsqueeze(1) @ fixed).squeeze(1) if drift else None
            dJ, gJ, chi2 = self.d_jastrow(r, e, x, chi)
            q = ratio * torch.exp(dJ)
            ok = unif[t] < q * q
            if drift:
                drifts.append(torch.stack([(v.squeeze(1) * y).sum(1) for v in out[1]], -1) / ratio.unsqueeze(1) + gJ)
            ratios.append(q)
            count += ok.to(torch.int32)
            m = ok.unsqueeze(1)
            if not pf:
                f = torch.where(ok, 1.0 / ratio, torch.zeros_like(ratio))
                if s == 0:
                    left = (row.unsqueeze(1) @ inv).squeeze(1)
                    left[:, e] -= 1.0
                    inv = inv - (col * f.unsqueeze(1)).unsqueeze(2) * left.unsqueeze(1)
                else:
                    left = (inv @ row.unsqueeze(2)).squeeze(2)
                    left[:, e - self.nu] -= 1.0
                    inv = inv - left.unsqueeze(2) * (col * f.unsqueeze(1)).unsqueeze(1)
            r[:, e] = torch.where(m, x, r[:, e])
            psi[:, e] = torch.where(m, new, psi[:, e])
            if self.LJ:
                chi = torch.where(ok[:, None, None], chi2, chi)
        return r, count, ratios, drifts

    def log_psi(self, r):
        la, sign = self.logdet(self.matrix(self._basis(r, self.kind, self.zeta, False)[0]))
        return la + self.jastrow(r)[0], sign


def _mul(a, b):
    """High and low words of a 32 x 32 bit product."""
    p = a * np.uint64(b)
    return p >> np.uint64(32), p & np.uint64(0xFFFFFFFF)


def _philox(seed, member, walkers, step, sigma):
    """Displacements and acceptance uniforms of one step: Philox4x32-10, counter (step, walker, member << 16 | block)."""
    out, m32 = [], np.uint64(0xFFFFFFFF)
    for blk in range(3):
        c = [np.full(walkers, v, np.uint64) for v in (step & 0xFFFFFFFF, step >> 32, 0, (member << 16) | blk)]
        c[2] = np.arange(walkers, dtype=np.uint64)
        k = [seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF]
        for _ in range(10):
            (h0, l0), (h1, l1) = _mul(c[0], 0xD2511F53), _mul(c[2], 0xCD9E8D57)
            c = [(h1 ^ c[1] ^ np.uint64(k[0])) & m32, l1, (h0 ^ c[3] ^ np.uint64(k[1])) & m32, l0]
            k = [(k[0] + 0x9E3779B9) & 0xFFFFFFFF, (k[1] + 0xBB67AE85) & 0xFFFFFFFF]
        out.append([(((c[i] << np.uint64(32)) | c[i + 1]) >> np.uint64(11)).astype(np.float64) * 2.0 ** -53 for i in (0, 2)])
    (u0, v0), (u1, v1), (u, _) = out
    a, b = np.sqrt(-2.0 * np.log1p(-u0)), np.sqrt(-2.0 * np.log1p(-u1))
    return sigma * np.stack([a * np.cos(2 * np.pi * v0), a * np.sin(2 * np.pi * v0), b * np.cos(2 * np.pi * v1)], -1), u


def _hops(X, case, r, xi, part):
    """One lattice iteration at r: hop ratios, the Green's function terms and the continuous-time step."""
    Wk, N = r.shape[:2]
    ev = X.in_parts(r, part)
    d = torch.sqrt(((r.unsqueeze(2) - X.R) ** 2).sum(-1))
    a = torch.full((Wk, N), case["a"], dtype=F64, device=X.dev)
    if case["a_valence"] > 0:
        a = torch.where((d < 0.8853 * X.Z ** (-1.0 / 3.0)).any(-1), a, torch.full_like(a, case["a_valence"]))
    step = torch.zeros(6, 3, dtype=F64, device=X.dev)
    for k in range(6):
        step[k, k // 2] = 1.0 - 2.0 * (k % 2)
    up = X._up()
    same = (up.unsqueeze(0) == up.unsqueeze(1))                       # [N, N]
    off = 1.0 - torch.eye(N, dtype=F64, device=X.dev)
    ratios = []
    for q in range(0, Wk, part):
        rr, yy, aa = r[q:q + part], ev["y"][q:q + part], a[q:q + part]
        cols = []
        for k in range(6):
            x = rr + aa.unsqueeze(-1) * step[k]
            det = (X._basis(x, X.kind, X.zeta, False)[0] * yy).sum(-1)
            dJ = 0.0
            for p, sg in ((x, 1.0), (rr, -1.0)):
                dn = p.unsqueeze(2) - X.R
                de = p.unsqueeze(2) - rr.unsqueeze(1)
                v = X._radial((de * de).sum(-1) + (1.0 - off), same)[0]
                dJ = dJ + sg * (X._one_body((dn * dn).sum(-1))[0].sum(-1) + (v * off).sum(-1))
            cols.append(det * torch.exp(dJ))
        ratios.append(torch.stack(cols, -1))
    ratios = torch.cat(ratios)
    ia2 = 1.0 / (a * a)
    lap = (ia2.unsqueeze(-1) * (ratios - 1.0)).sum((1, 2))
    H = (-0.5 * ia2).unsqueeze(-1)
    flip = ratios < 0
    vsf = torch.where(flip, H * ratios, torch.zeros_like(ratios)).sum((1, 2))
    G = -torch.where(flip, -case["gamma"] * H, H) * ratios
    escape = G.sum((1, 2))
    shift = 0.5 * (lap + 2.0 * ev["e_kin"])
    diag = 3.0 * ia2.sum(-1) + (ev["e_loc"] - ev["e_kin"]) + shift + (1.0 + case["gamma"]) * vsf
    terms = torch.stack([ev["e_loc"], ev["e_kin"], lap, shift, vsf, escape, diag], 1)
    stay = -torch.log1p(-xi[:, 0]) / escape
    hop = stay < case["tau"]
    left = torch.where(hop, case["tau"] - stay, torch.zeros_like(stay))
    weight = torch.exp(-torch.where(hop, stay, torch.full_like(stay, case["tau"])) * ev["e_loc"])
    k = (G.flatten(1).cumsum(1) <= (xi[:, 1] * escape).unsqueeze(1)).sum(1).clamp(max=6 * N - 1)
    b = torch.arange(Wk, device=X.dev)
    nxt = r.clone()
    nxt[b, k // 6] += torch.where(hop, a[b, k // 6], torch.zeros_like(stay)).unsqueeze(1) * step[k % 6]
    return ratios, terms, nxt, weight, left


def exact(case, seed):
    dev = torch.device("cuda:0")
    kind = case["kind"]
    t = lambda a: torch.tensor(a, device=dev)  # noqa: E731
    if kind == "sr":
        O, e = _sr_inputs(case, seed)
        D = O - O.mean(0)
        f = -2.0 * (D.T @ e) / len(O)
        S = D.T @ D / len(O)
        S.diagonal().mul_(1.0 + case["eps"])
        return dict(delta=torch.linalg.solve(S.cpu(), f.cpu()), force=f)
    x = _host_inputs(case, seed)
    if kind == "multi":
        out = {}
        for i, s in enumerate(x.systems):
            X = _Exact(s, dev)
            draws = [_philox(x.key, i, case["walkers"], k, 0.3) for k in range(case["moves"])]
            r, _, _, _ = X.chain(t(x.r0[i]), t(np.stack([d for d, _ in draws])), t(np.stack([u for _, u in draws])))
            la, sign = X.log_psi(r)
            out["%02d" % i] = dict(r=r, logabs=la, sign=sign)
        return out
    X = _Exact(x.s, dev)
    N, L = X.N, len(x.s.zeta)
    part = max(1, int(4e8 // (N * L * 8)))                            # walkers at once: temporaries of some hundred MB
    r = t(x.r0)
    only = lambda ev, keys: {k: ev.get(k) for k in keys}  # noqa: E731
    if kind == "eval":
        return only(X.in_parts(r, part), ("logabs", "sign", "drift", "e_kin", "e_loc", "status"))
    if kind == "vmc":
        r, _, _, _ = X.chain(r, t(x.disp), t(x.unif))
        return dict(only(X.in_parts(r, part), ("logabs", "sign", "drift", "e_kin", "e_loc", "status")), r=r, count=None)
    if kind == "moves":
        r, _, q, d = X.chain(r, t(x.disp), t(x.unif), drift=True)
        return dict(ratios=torch.stack(q), drifts=torch.stack(d), r=r, logabs=X.log_psi(r)[0], status=None)
    if kind == "lrdmc":
        ratios, terms, nxt, weight, left = _hops(X, case, r, t(x.xi), part)
        return dict(only(X.in_parts(nxt, part), ("logabs", "sign", "e_kin", "e_loc", "status")), ratios=ratios,
                    terms=terms, r=nxt, hop=None, weight=weight, left=left)
    if kind == "grad":
        names = ("R", "zeta", "lam", "jas")
        for k in names:
            getattr(X, k).requires_grad_(True)
        r.requires_grad_(True)
        part = max(1, part // 8)
        gl, ge = t(x.gl), t(x.ge)
        la, el = [], []
        for q in range(0, len(r), part):
            ev = X.evaluate(r[q:q + part])
            torch.autograd.backward([ev["logabs"], ev["e_loc"]], [gl[q:q + part], ge[q:q + part]])
            la.append(ev["logabs"].detach())
            el.append(ev["e_loc"].detach())
        return dict(logabs=torch.cat(la), e_loc=torch.cat(el), r=r.grad, **{k: getattr(X, k).grad for k in names})
    # logder: every walker its own copy of the parameters
    Wk = len(r)
    own = ["R", "zeta", "lam", "jas"] + (["U"] if X.U.shape[1] else []) + (["jzeta", "j1", "j3"] if X.LJ else [])
    for k in own:
        v = getattr(X, k)
        setattr(X, k, v.expand(Wk, *v.shape).contiguous().requires_grad_(True))
    r.requires_grad_(True)
    la, _ = X.log_psi(r)
    la.sum().backward()
    name = dict(U="unpaired", jzeta="jb_zeta", j1="j1_inh")
    out = {name.get(k, k): getattr(X, k).grad for k in own}
    if X.LJ:
        g = out["j3"]
        out["j3"] = torch.cat([0.5 * (g[:, :2] + g[:, :2].transpose(-1, -2)), g[:, 2:]], 1)
    return dict(out, r=r.grad)
