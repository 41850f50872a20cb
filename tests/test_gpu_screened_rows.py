"""Screened proposals past the resident sizes, and QMC_REFINED ones of small systems:
row counts around a workgroup's (128 or 256 rows, by the number of walkers) and
around the lanes a column takes, odd ones among them, kept lists longer than a block
of 1024; ratios of both spins against plain torch, with the first and last walker
repeated through the set."""
import pytest
import torch

from gpu_util import need_gpu
from oracle import jagp as O
from test_gpu_chain import _system
from test_gpu_small_ratios import EPS, _terms
from workloads import configs as C

pytestmark = pytest.mark.gpu


# (seeds of systems whose W is regular: the test is of the stream)
@pytest.mark.parametrize("n_up,n_dn,shells,walkers,precision,seed", [
    (3, 2, (0, 0, 1), 3, "QMC_REFINED", 1),
    (17, 16, (0, 0, 1), 300, "QMC_REFINED", 1),
    (33, 32, (0, 0, 1), 5, "QMC_REFINED", 5),
    (129, 129, (0, 0, 1), 4, "QMC_FP64", 4),
    (129, 128, (0, 0, 1), 256, "QMC_FP64", 8),
    (160, 158, (0, 0, 1), 256, "QMC_REFINED", 4),
    (161, 161, (0, 0, 1), 40, "QMC_REFINED", 6),
    (257, 256, (0, 0, 1), 4, "QMC_FP64", 3),
    (257, 257, (0, 0, 1), 128, "QMC_REFINED", 6),
    (140, 140, (0,) * 5 + (1,) * 2, 4, "QMC_FP64", 2),
    (24, 24, (0,) * 30 + (1,) * 18, 3, "QMC_FP64", 1)])
def test_ratios(n_up, n_dn, shells, walkers, precision, seed):
    P = need_gpu()
    s = _system(n_up, n_dn, shells, 16, seed=seed)
    few = 3
    r = torch.tensor(C.random_positions(81, s, few))
    at = torch.arange(walkers) % few
    sy = O.from_workload_system(s)
    cond = torch.linalg.cond(O.evaluate(sy, r, with_intermediates=True)["W"])
    wk = P.Walkers(P.JAGPSystem(s, precision=getattr(P, precision)), walkers, adjoint=False)
    wk.eval_batch(r[at].contiguous().cuda())
    g = torch.Generator().manual_seed(7)
    for e in (0, n_up - 1, n_up, n_up + n_dn - 1):
        rn = r[:, e] + 0.4 * torch.randn(few, 3, generator=g, dtype=torch.float64)
        R, E, dJ = _terms(sy, r, e, rn)
        q = wk.propose(e, rn[at].contiguous().cuda()).cpu()
        want = R * torch.exp(dJ)
        # the order of the sums, and W^{-1} on both sides: eps cond(W) a term; QMC_REFINED's
        # rows and what it leaves out: 1e-13 in their place
        unit = EPS if precision == "QMC_FP64" else 1e-13
        tol = (len(s.lam) + cond[:, None]).amax(1) * 8 * unit * E * torch.exp(dJ)
        assert (tol <= 1e-2 * want.abs()).all()
        assert ((q - want[at]).abs() <= tol[at]).all(), (e, (q / want[at] - 1).abs().max())
