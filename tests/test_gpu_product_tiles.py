"""E_loc of evaluations at the edges of the FP64 products' three tiles (64 x 64,
32 x 64 and 32 x 32, by the sizes and the number of walkers), unpaired columns and a
banded Lambda among them, on systems whose W is regular (cond < 1e6), so that every
case is held to the FP64 bar of 1e-10."""
import numpy as np
import pytest
import torch

from gpu_util import need_gpu, rel_err
from oracle import jagp as O
from test_gpu_chain import _system
from workloads import configs as C


def _regular(n_up, n_dn, shells, band, seed):
    s = _system(n_up, n_dn, shells, 32, seed=seed)
    if band:   # zero tiles of Lambda are skipped
        L = len(s.zeta)
        d = np.abs(np.arange(L)[:, None] - np.arange(L)[None, :])
        s.lam = np.where(d < 40, s.lam, 0.0) + np.eye(L)
    r = torch.tensor(C.random_positions(61, s, 3))
    return s, r, O.evaluate(O.from_workload_system(s), r, with_intermediates=True)


CASES = [(27, 25, (0, 0, 0, 1, 1), False, 1, 260), (33, 32, (0, 0, 0, 1), False, 4, 130),
         (64, 63, (0, 0, 0, 1), False, 4, 70), (65, 65, (0, 0, 0, 1), True, 4, 40),
         (100, 99, (0, 0, 0, 1), False, 5, 24), (129, 129, (0, 0, 1), True, 23, 12)]


@pytest.mark.gpu
@pytest.mark.parametrize("n_up,n_dn,shells,band,seed,many", CASES)
def test_local_energy_at_the_tiles_edges(n_up, n_dn, shells, band, seed, many):
    P = need_gpu()
    s, r, ref = _regular(n_up, n_dn, shells, band, seed)
    assert torch.linalg.cond(ref["W"]).max().item() < 1e6
    sysh = P.JAGPSystem(s)
    for Wk in (3, many):
        out = P.Walkers(sysh, Wk, adjoint=False).eval_batch(r[torch.arange(Wk) % 3].contiguous().cuda())
        for k in ("logabs", "e_kin", "e_loc"):
            assert rel_err(out[k][:3].cpu(), ref[k]).max().item() <= 1e-10, (Wk, k)
