"""Proposals with a drift in one launch (up to 24 KiB of rows, and past it in three),
and the one-launch list of the rows moved since they were built (up to 8192 rows a
spin), at the sizes on both sides of their rules.
"""
import numpy as np
import pytest
import torch

from gpu_util import need_gpu, rel_err
from oracle import jagp as O
from test_gpu_chain import _system
from workloads import configs as C

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["QMC_FP64", "QMC_MIXED", "QMC_W_FP32", "QMC_MIXED_BF16", "QMC_REFINED"])
@pytest.mark.parametrize("n_up,n_dn,shells", [(1, 1, (0,)), (2, 1, (0, 0, 1)), (9, 8, (0, 0, 1)), (24, 24, (0, 0, 1)),
                                              (25, 24, (0, 0, 0, 0, 1))])
def test_drift_proposals(n_up, n_dn, shells, precision):
    # against the evaluation at the moved positions, at the precision of the rows
    P = need_gpu()
    s = _system(n_up, n_dn, shells, 64, jastrow=n_up == 9)
    N, Wk = n_up + n_dn, 3
    r = torch.tensor(C.random_positions(71, s, Wk))
    wk = P.Walkers(P.JAGPSystem(s, precision=getattr(P, precision)), Wk, adjoint=False)
    wk.eval_batch(r.cuda())
    sy = O.from_workload_system(s)
    ref0 = O.evaluate(sy, r, with_intermediates=True)
    eps = {"QMC_FP64": 2.0 ** -52, "QMC_REFINED": 2.0 ** -46, "QMC_MIXED_BF16": 2.0 ** -8}.get(precision, 2.0 ** -23)
    for e in {0, n_up - 1, n_up, N - 1}:
        rn = r.clone()
        rn[:, e] += torch.tensor([0.3, -0.2, 0.1])
        q, d = wk.propose(e, rn[:, e].cuda().contiguous(), drift=True)
        ref = O.evaluate(sy, rn)
        want = ref["sign"] * ref0["sign"] * torch.exp(ref["logabs"] - ref0["logabs"])
        # rows rounded to eps: the ratio is a sum of L products over the inverse's column
        W, A = ref0["W"], ref0["A"]
        k = e if e < n_up else e - n_up
        col = A[:, :, k] if e < n_up else A[:, k, :]
        L = len(s.zeta)
        scale = col.abs().sum(1) * W.abs().amax((1, 2)) * L
        tol = 8 * eps * scale.max().item() * max(1.0, torch.exp(ref["J"] - ref0["J"]).max().item() if "J" in ref else 4.0)
        assert ((q.cpu() - want).abs().max().item()) <= max(tol, 1e-10)
        if precision in ("QMC_FP64", "QMC_REFINED"):
            dref = ref["drift"][:, e]
            assert ((d.cpu() - dref).abs() / dref.abs().clamp(min=1.0)).max().item() <= 1e-8 * max(1.0, 1e-6 * scale.max().item())


@pytest.mark.parametrize("precision", ["QMC_FP64", "QMC_REFINED"])
@pytest.mark.parametrize("n_up,n_dn,Wk", [(26, 25, 3), (26, 26, 315), (26, 25, 316), (27, 1, 64)])
def test_rows_moved_since_the_last_build(n_up, n_dn, Wk, precision):
    # the second evaluation builds only the moved rows: bitwise a fresh one
    P = need_gpu()
    s = _system(n_up, n_dn, (0, 0, 0, 1, 1), 64)
    N = n_up + n_dn
    g = torch.Generator().manual_seed(3)
    r = torch.tensor(C.random_positions(73, s, 8)).repeat(-(-Wk // 8), 1, 1)[:Wk].contiguous()
    r += 0.1 * torch.rand(r.shape, generator=g, dtype=torch.float64)
    sysh = P.JAGPSystem(s, precision=getattr(P, precision))
    wk = P.Walkers(sysh, Wk, adjoint=False)
    wk.eval_batch(r.cuda())
    for frac in (0.0, 0.3, 1.0):
        mv = torch.rand(Wk, N, generator=g) < frac
        r = torch.where(mv[:, :, None], r + 0.05 * torch.randn(r.shape, generator=g, dtype=torch.float64), r)
        if frac == 0.3:   # the first and the last row, one coordinate
            r[0, 0, 2] += 0.01
            r[-1, -1, 0] -= 0.01
        out = wk.eval_batch(r.cuda())
        fresh = P.Walkers(sysh, Wk, adjoint=False)
        ref = fresh.eval_batch(r.cuda())
        for k in ("logabs", "sign", "e_kin", "e_loc", "drift"):
            assert torch.equal(out[k], ref[k]), (frac, k)
        assert torch.equal(wk.read(P.STATE_W), fresh.read(P.STATE_W))
