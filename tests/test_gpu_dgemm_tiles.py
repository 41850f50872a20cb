"""The FP64 products' tiles (32 x 32 to 128 x 64, chosen by the sizes and the
number of walkers): electron counts at the tiles' edges, odd and even leading
dimensions, unpaired columns, a banded Lambda.  A walker's evaluation does not
depend on how many others share the launch, bitwise, whatever tiles that takes;
three walkers against the oracle at the FP64 bars (1e-10 on log|Psi| and E_loc).
"""
import numpy as np
import pytest
import torch

from gpu_util import need_gpu, rel_err
from oracle import jagp as O
from workloads import configs as C

pytestmark = pytest.mark.gpu


def _system(n_up, n_dn, shells, band):
    rng = np.random.default_rng(5 + 1000 * n_up + n_dn)
    N = n_up + n_dn
    A = max(2, (N + 1) // 2)
    R = C._place_nuclei(rng, A, (60.0 * N) ** (1 / 3) + 3.0)
    center, l, m, zeta = C._shell_basis(rng, A, list(shells), 0.1, 10.0)
    L = len(zeta)
    lam = C._sym_gaussian(rng, L, 1.0 / L)
    if band:   # zero tiles of Lambda are skipped
        d = np.abs(np.arange(L)[:, None] - np.arange(L)[None, :])
        lam = np.where(d < 40, lam, 0.0) + np.eye(L)
    return C.System(name="tiles", R=R, Z=np.full(A, 2.0), center=center, l=l, m=m, zeta=zeta,
                    radial=np.zeros(L, np.int32), lam=lam, n_up=n_up, n_dn=n_dn,
                    unpaired=rng.standard_normal((L, n_up - n_dn)) / np.sqrt(L), j1_form=2, j1_b=np.ones(A),
                    j2_form=1, j2=np.array([1.0, 1.0]), refresh_every=32)


@pytest.mark.parametrize("n_up,n_dn,shells,band,many", [
    (27, 25, (0, 0, 0, 1, 1), False, 260), (33, 32, (0, 0, 0, 1), False, 130), (64, 63, (0, 0, 1), False, 70),
    (65, 65, (0, 0, 1), True, 40), (100, 99, (0, 0, 0, 1), False, 24), (129, 129, (0, 0, 1), True, 12)])
def test_evaluation_does_not_depend_on_the_tiles(n_up, n_dn, shells, band, many):
    P = need_gpu()
    s = _system(n_up, n_dn, shells, band)
    sysh = P.JAGPSystem(s)
    r = torch.tensor(C.random_positions(61, s, many)).cuda()
    res = []
    for Wk in (many, 3, 1):
        wk = P.Walkers(sysh, Wk, adjoint=False)
        out = wk.eval_batch(r[:Wk].contiguous())
        res.append((out["logabs"], out["e_loc"], out["drift"], wk.read(P.STATE_W), wk.read(P.STATE_AINV)))
    for x in res[1:]:
        k = len(x[0])
        for a, b in zip(res[0], x):
            assert torch.equal(a[:k], b)
    ref = O.evaluate(O.from_workload_system(s), r[:3].cpu(), with_intermediates=True)
    assert rel_err(res[1][0].cpu(), ref["logabs"]).max().item() <= 1e-10
    W = res[1][3].cpu()
    assert ((W - ref["W"]).abs().max() / ref["W"].abs().max()).item() <= 1e-12
    if torch.linalg.cond(ref["W"]).max().item() < 1e6:
        assert rel_err(res[1][1].cpu(), ref["e_loc"]).max().item() <= 1e-10
