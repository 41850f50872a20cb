"""The inverse with its columns split between four waves (17 to 96 rows): row counts
at the ends of its widths, one and two rows a lane, and the walker count at which
two waves take over past 64 rows.  Bars as for every FP64 evaluation: |W A - I| below
1e-9, log|Psi| 1e-10 relative; a walker's inverse does not depend on the count.
"""
import pytest
import torch

from gpu_util import need_gpu, rel_err
from oracle import jagp as O
from test_gpu_chain import _system
from workloads import configs as C

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_up,n_dn,many", [(17, 17, 0), (24, 23, 0), (25, 25, 0), (40, 40, 0), (57, 57, 0), (64, 63, 0),
                                            (65, 65, 513), (72, 72, 0), (88, 88, 513), (89, 89, 0), (96, 96, 513)])
def test_four_wave_inverse(n_up, n_dn, many):
    P = need_gpu()
    s = _system(n_up, n_dn, (0, 0, 0, 1, 1), 32)
    sysh = P.JAGPSystem(s)
    r = torch.tensor(C.random_positions(83, s, 4))
    r[1, 1] = r[1, 0]   # two equal rows: singular
    rows = r.repeat(-(-many // 4), 1, 1)[:many] if many else r
    res = []
    for x in (r, rows):
        wk = P.Walkers(sysh, len(x), adjoint=False)
        out = wk.eval_batch(x.cuda())
        res.append((out, wk.read(P.STATE_W)[:4].cpu(), wk.read(P.STATE_AINV)[:4].cpu()))
    (out, W, A), (out2, W2, A2) = res
    ok = [0, 2, 3]
    assert torch.equal(W, W2) and torch.equal(A[ok], A2[ok])
    assert rel_err(out2["logabs"].cpu()[ok], out["logabs"].cpu()[ok]).max().item() <= 1e-14
    st = out["status"].cpu()
    assert (st[ok] == 0).all() and st[1] != 0
    ref = O.evaluate(O.from_workload_system(s), r[ok], with_intermediates=True)
    assert rel_err(out["logabs"].cpu()[ok], ref["logabs"]).max().item() <= 1e-10
    assert torch.equal(out["sign"].cpu()[ok], ref["sign"])
    eye = torch.eye(n_up, dtype=torch.float64)
    cond = torch.linalg.cond(ref["W"])
    for i, w in enumerate(ok):
        assert (W[w] @ A[w] - eye).abs().max().item() <= max(1e-9, 1e-14 * cond[i].item())
