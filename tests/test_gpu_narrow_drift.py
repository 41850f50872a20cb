"""Proposals with a drift at every storage of the P rows: the ratio and the drift
against the FP64 oracle within what rounding the rows gives, and one launch against
three, bit for bit, where the number of walkers decides between them (rows of 16 to
24 KiB)."""
import numpy as np
import pytest
import torch

from gpu_util import need_gpu
from oracle import jagp as O
from test_gpu_chain import _system
from workloads import configs as C

# unit roundoff of what is stored
ROUND = {"QMC_FP64": 2.0 ** -53, "QMC_W_FP32": 2.0 ** -24, "QMC_MIXED": 2.0 ** -24, "QMC_MIXED_BF16": 2.0 ** -9}


def _spread(F, x, lam, U, D, y, u):
    """Root mean square, over walkers, of what one relative rounding of at most u in
    each element of F, Lambda, U, D and of the rows D Lambda^T, and sums of L products
    rounded in FP32 (FP64 for FP64 rows), do to sum_ij x_i (F [Lambda D^T | U])_ij y_j."""
    L, nd = lam.shape[0], D.shape[1]
    yd, yu = y[:, :nd], y[:, nd:]
    rows = D @ lam.T                                        # [w, j, l]
    q = torch.einsum('wj,wjl->wl', yd, rows) + yu @ U.T
    f = torch.einsum('wi,wil->wl', x, F)
    d = torch.einsum('wj,wjl->wl', yd, D)
    acc = (D ** 2) @ (lam.T ** 2)                            # partial sums of a row's element
    s = torch.einsum('wi,wil,wl->w', x ** 2, F ** 2, q ** 2)
    s = s + torch.einsum('wl,lm,wm->w', f ** 2, lam ** 2, d ** 2)
    s = s + torch.einsum('wj,wjl,wl->w', yd ** 2, D ** 2, (f @ lam) ** 2)
    s = s + torch.einsum('wj,wjl,wl->w', yd ** 2, rows ** 2 + L * (min(u, 2.0 ** -24) / u) ** 2 * acc, f ** 2)
    s = s + torch.einsum('wk,lk,wl->w', yu ** 2, U ** 2, f ** 2)
    return u * s.sqrt()


def _bounds(s, sy, r, rn, e, precision):
    """ratio, drift and how far rounded rows may take them from these: R and grad R are
    sums f Lambda D^T A_e, with f the functions or their gradient at r', to which each
    rounding adds independently (_spread; eight of its root mean squares).  FP32 products
    of the evaluation change W too, and so R by f Lambda D^T A dW A_e."""
    nu = s.n_up
    u = ROUND[precision]
    ref, new = O.evaluate(sy, r, with_intermediates=True), O.evaluate(sy, rn, with_intermediates=True)
    A, pu, pd = ref["A"], ref["Phi"][:, :nu], ref["Phi"][:, nu:]
    if e < nu:
        lam, D, U, col = sy.lam, pd, sy.unpaired, A[:, :, e]
    else:
        lam, D, U, col = sy.lam.T, pu, sy.unpaired[:, :0], A[:, e - nu]
    rows = torch.cat([D @ lam.T, U.T.expand(len(r), -1, -1)], 1)
    one = torch.ones(len(r), 1, dtype=torch.float64)

    def err(f):   # f [Wk, L]: a functional of the moved electron
        d = _spread(f[:, None], one, lam, U, D, col, u)
        if precision == "QMC_W_FP32":
            v = torch.einsum('wjl,wl->wj', rows, f)
            if e < nu:   # v A is a row over the up electrons, A_e over the columns
                d = d + _spread(pu, torch.einsum('wj,wji->wi', v, A), sy.lam, sy.unpaired, pd, col, u)
            else:
                d = d + _spread(pu, col, sy.lam, sy.unpaired, pd, torch.einsum('wji,wi->wj', A, v), u)
        return 8 * d

    R = torch.einsum('wjl,wl,wj->w', rows, new["Phi"][:, e], col)
    dR = err(new["Phi"][:, e])
    grad = new["gradPhi"][:, e]
    g = torch.einsum('wjl,wlx,wj->wx', rows, grad, col)
    dg = torch.stack([err(grad[:, :, x]) for x in range(3)], 1)
    J = torch.exp(new["J"] - ref["J"])
    want = new["sign"] * ref["sign"] * torch.exp(new["logabs"] - ref["logabs"])
    assert torch.allclose(R * J, want, rtol=1e-9, atol=0) and (dR < 0.5 * R.abs()).all()
    dD = (dg + (g / R[:, None]).abs() * dR[:, None]) / (R.abs() - dR)[:, None]
    # and what FP64 itself gives through an inverse of this condition
    fp64 = 64 * 2.0 ** -53 * torch.linalg.cond(ref["W"])
    return want, new["drift"][:, e], dR * J + fp64 * want.abs(), dD + (fp64 * (1 + new["drift"][:, e].norm(dim=1)))[:, None]


def _inputs(s, Wk=3, step=0.1):
    r = torch.tensor(C.random_positions(71, s, Wk))
    def moved(e):
        rn = r.clone()
        rn[:, e] += step * torch.tensor([0.9, -0.6, 0.3])
        return rn
    return r, moved


SHAPES = [(2, 1, (0, 0, 1), 38), (5, 5, (0, 0, 1), 32), (9, 8, (0, 0, 1), 4), (16, 16, (0, 0, 1, 1), 19),
          (24, 24, (0, 0, 0, 0, 0, 1), 5)]


@pytest.mark.gpu
@pytest.mark.parametrize("precision", list(ROUND))
@pytest.mark.parametrize("n_up,n_dn,shells,seed", SHAPES)
def test_ratio_and_drift_of_stored_rows(n_up, n_dn, shells, seed, precision):
    P = need_gpu()
    s = _system(n_up, n_dn, shells, 64, seed=seed)
    sy = O.from_workload_system(s)
    r, moved = _inputs(s)
    wk = P.Walkers(P.JAGPSystem(s, precision=getattr(P, precision)), len(r), adjoint=False)
    wk.eval_batch(r.cuda())
    for e in sorted({0, n_up - 1, n_up, n_up + n_dn - 1}):
        want, drift, tq, td = _bounds(s, sy, r, moved(e), e, precision)
        q, d = wk.propose(e, moved(e)[:, e].cuda().contiguous(), drift=True)
        assert ((q.cpu() - want).abs() <= tq).all(), e
        assert ((d.cpu() - drift).abs() <= td).all(), e


@pytest.mark.gpu
@pytest.mark.parametrize("precision,n,L", [("QMC_FP64", 20, 120), ("QMC_W_FP32", 24, 192), ("QMC_MIXED", 24, 192),
                                           ("QMC_MIXED_BF16", 32, 320)])
def test_one_launch_equals_three(precision, n, L):
    P = need_gpu()
    s = _system(n, n, (0,) * (L // n) + (() if L % n == 0 else (0,)), 64)
    sysh = P.JAGPSystem(s, precision=getattr(P, precision))
    r, moved = _inputs(s, 4)
    few, many = P.Walkers(sysh, 4, adjoint=False), P.Walkers(sysh, 8196, adjoint=False)
    few.eval_batch(r.cuda())
    many.eval_batch(r.repeat(2049, 1, 1).cuda())
    for item in (P.STATE_W, P.STATE_AINV):
        assert torch.equal(many.read(item)[:4], few.read(item))
    for e in (0, n - 1, n, 2 * n - 1):
        rn = moved(e)[:, e].contiguous()
        q, d = few.propose(e, rn.cuda(), drift=True)
        qm, dm = many.propose(e, rn.repeat(2049, 1).cuda(), drift=True)
        assert torch.equal(qm, q.repeat(2049)) and torch.equal(dm, d.repeat(2049, 1)), e
