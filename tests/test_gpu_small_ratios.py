"""QMC_FP64 moves whose ratio is far below one (an electron moved out of the
molecule, without a node in between): the ratio keeps its digits, and accepting
such a move leaves a finite log|Psi| and a usable W, by the resident runs, the
single proposals of both resident forms and the per-move path (past 128 rows, past
1024 functions, wide Jastrow bases).  (The delayed form of the inverse takes 1 / R
from a difference of sums of order one, so its W^{-1} holds again from the next
refresh on: the per-move path is asked for log|Psi| and the moves after a refresh.)

The reference is R = sum_j c_j sum_mu P_j[mu] psi_mu(r') in plain torch.  A ratio
summed in any order is within (L + n) eps sum_j |c_j| sum_mu |P_j[mu] psi_mu| of
it, and both sides' c (an inverse) differ by a few n eps cond(W) of themselves,
held to 1e-9.  log|Psi| after an accept adds log|R|, so its absolute bar is the
ratio's relative one beside the usual 1e-10 of log|Psi|.
"""
import numpy as np
import pytest
import torch

from gpu_util import need_gpu, rel_err
from oracle import jagp as O
from test_gpu_chain import _system as _chain_system
from test_gpu_screened_fp64 import _system as _plain_system
from workloads import configs as C

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -52
DIST = (0.3, 5.0, 9.0, 14.0, 19.0, 24.0, 30.0, 36.0)   # bohr past the cube's far corner


def _outside(s, d):   # (d < 0: past the near corner)
    far = np.asarray(s.R).max(0) + d / 3 ** 0.5 if d > 0 else np.asarray(s.R).min(0) + d / 3 ** 0.5
    return torch.tensor(np.broadcast_to(far, (1, 3)).copy())


def _terms(sy, r, e, rn):
    """(R, sum of the terms' magnitudes, dJ) of electron e to rn, from plain arrays."""
    nu = sy.n_up
    ref = O.evaluate(sy, r, with_intermediates=True)
    phi, A = ref["Phi"], ref["A"]
    psi = O.agp_basis(sy, torch.cat([rn[:, None], r[:, 1:]], 1))[0][:, 0]
    if e < nu:
        P = torch.cat([phi[:, nu:] @ sy.lam.T, sy.unpaired.T.expand(r.shape[0], -1, -1)], 1)
        c = A[:, :, e]
    else:
        P = phi[:, :nu] @ sy.lam
        c = A[:, e - nu, :]
    R = torch.einsum("wj,wjm,wm->w", c, P, psi)
    E = torch.einsum("wj,wjm,wm->w", c.abs(), P.abs(), psi.abs())
    r2 = r.clone()
    r2[:, e] = rn
    dJ = O.evaluate(sy, r2)["J"] - ref["J"]
    return R, E, dJ


CASES = [
    (lambda: _plain_system(11, 9), "small resident form, single moves per move"),
    (lambda: _plain_system(33, 32), "large resident form"),
    (lambda: _plain_system(66, 65), "large resident form, two rows a lane"),
    (lambda: _chain_system(30, 30, (0, 0, 0, 0, 0, 1, 1, 2), 16), "large resident form, two functions a thread"),
    (lambda: _chain_system(34, 33, (0, 0, 0, 1), 16, True), "large resident form with a Jastrow basis"),
    (lambda: _chain_system(65, 65, (0, 0, 0, 1), 16, True), "a wide Jastrow basis: per move"),
    (lambda: _plain_system(131, 129), "past 128 rows: per move"),
    (lambda: _chain_system(24, 24, (0,) * 14 + (1,) * 10, 16), "past 1024 functions: per move, 1024 threads"),
]
SINGLE, RUN = (1, 2, 3, 4), (0, 1, 2, 3, 4)   # where W^{-1} itself is kept


@pytest.mark.parametrize("case", range(len(CASES)), ids=[c[1] for c in CASES])
def test_ratio_keeps_its_digits(case):
    P = need_gpu()
    s = CASES[case][0]()
    Wk = len(DIST)
    r = torch.tensor(C.random_positions(17, s, 1)).repeat(Wk, 1, 1)
    sy = O.from_workload_system(s)
    wk = P.Walkers(P.JAGPSystem(s), Wk, adjoint=False)
    rn = torch.cat([_outside(s, d) for d in DIST])
    for e in (0, s.n_up - 1, s.n_up, s.n_up + s.n_dn - 1):
        wk.eval_batch(r.cuda())
        R, E, dJ = _terms(sy, r, e, rn)
        q = wk.propose(e, rn.cuda()).cpu()
        qd = wk.propose(e, rn.cuda(), drift=True)[0].cpu()
        tol = (1e-9 + (len(s.lam) + s.n_up) * EPS * E / R.abs()) * (R * torch.exp(dJ)).abs()
        assert R.abs().min() < 1e-30 and (E / R.abs()).max() < 1e6   # what the case is for
        assert ((q - R * torch.exp(dJ)).abs() <= tol).all(), (q / (R * torch.exp(dJ)) - 1)
        assert ((q - qd).abs() <= tol).all()
        # accepted: log|Psi| follows, and the walker's state is that of an evaluation there
        wk.propose(e, rn.cuda())
        wk.accept(e, torch.ones(Wk, dtype=torch.uint8, device="cuda"))
        la, sg = wk.read(P.STATE_LOGABS).cpu(), wk.read(P.STATE_SIGN).cpu()
        r2 = r.clone()
        r2[:, e] = rn
        ref, rs = O.log_psi(sy, r2)
        assert ((la - ref).abs() <= 1e-10 * ref.abs().clamp(min=1) + tol / (R * torch.exp(dJ)).abs()).all(), la - ref
        assert torch.equal(sg, rs)
        if case in SINGLE:
            assert torch.isfinite(wk.read(P.STATE_AINV)).all()


@pytest.mark.parametrize("case", range(len(CASES)), ids=[c[1] for c in CASES])
def test_runs_take_such_moves(case):
    # electrons leave (u = 0 accepts any ratio but zero): the last of a spin, one at the
    # end, and where the inverse is kept one among ordinary moves, the other way (two of
    # a spin far out on one side would make W singular to ten digits)
    P = need_gpu()
    s = CASES[case][0]()
    Wk, n = 3, 12
    e0, leave = (s.n_up - 6) % (s.n_up + s.n_dn), {5: 24.0, n - 1: 30.0, **({2: -27.0} if case in RUN else {})}
    r = torch.tensor(C.random_positions(19, s, Wk))
    disp, unif = (torch.tensor(x) for x in C.chain_arrays(43, n, Wk))
    for t, d in leave.items():
        disp[t] = _outside(s, d) - r[:, (e0 + t) % (s.n_up + s.n_dn)]
        unif[t] = 0.0
    wk = P.Walkers(P.JAGPSystem(s), Wk, adjoint=False)
    wk.eval_batch(r.cuda())
    wk.vmc_steps(e0, disp.cuda(), unif.cuda())
    sy = O.from_workload_system(s)
    rf, ratios, acc = O.run_chain(sy, r, disp, unif, e_start=e0)
    assert acc[list(leave)].all() and ratios[list(leave)].abs().max() < 1e-16
    assert torch.equal(wk.read(P.STATE_R).cpu(), rf)
    la, ref = wk.read(P.STATE_LOGABS).cpu(), O.log_psi(sy, rf)[0]
    assert rel_err(la, ref).max().item() <= 1e-9
