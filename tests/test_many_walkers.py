"""More walkers than a grid's second dimension counts (65535): every launch of the
evaluation, the moves and the runs fits the device's limits (recorded, nothing
runs), and the last walkers' ratios are those of a small set (GPU)."""
import inspect

import numpy as np
import pytest
import torch

from gpu_util import need_gpu
from recorder import run
from test_gpu_chain import _system
from workloads import configs as C

# (the source alone: no torch in the recording process)
HEAD = inspect.getsource(_system)
SCRIPT = """
s = _system({n_up}, {n_dn}, {shells}, 16)
h = P.JAGPSystem(s, precision=P.{precision})
k = P.Walkers(h, {walkers}, adjoint=False)
def go():
    ok(lib.qmc_eval_batch(h.h, k.h, dev(1), dev(2), dev(3), dev(4), dev(5), dev(6), dev(7), None))
    for e in (0, {n_up}):
        for drift in (None, dev(4)):
            ok(lib.qmc_propose_move(h.h, k.h, e, dev(1), dev(2), drift, None))
            ok(lib.qmc_accept_move(h.h, k.h, e, dev(3), None, None))
    ok(lib.qmc_vmc_steps(h.h, k.h, 0, 40, dev(1), dev(2), dev(3), None))
out = [x for x in kernels(go)]
"""
WIDE = (0,) * 260   # 520 functions of two nuclei


@pytest.mark.parametrize("precision", ["QMC_FP64", "QMC_REFINED", "QMC_MIXED"])
@pytest.mark.parametrize("n_up,n_dn,shells", [(2, 2, (0, 0, 1)), (1, 1, WIDE), (40, 40, (0, 0, 0, 1))])
def test_launches_fit_the_device(n_up, n_dn, shells, precision):
    out = run(HEAD + SCRIPT.format(n_up=n_up, n_dn=n_dn, shells=shells, walkers=65600, precision=precision))
    assert len(out) > 10
    for name, grid, block in out:
        assert grid[0] < 2 ** 31 and grid[1] <= 65535 and grid[2] <= 65535, (name, grid)
        assert block[0] * block[1] * block[2] <= 1024, (name, block)


@pytest.mark.gpu
def test_ratios_of_the_last_walkers():
    P = need_gpu()
    s = _system(1, 1, WIDE, 16)
    Wk, few = 65600, 16
    r = torch.tensor(C.random_positions(3, s, few)).cuda()
    sysh = P.JAGPSystem(s)
    many, some = P.Walkers(sysh, Wk, adjoint=False), P.Walkers(sysh, few, adjoint=False)
    many.eval_batch(r.repeat(Wk // few, 1, 1).contiguous())
    some.eval_batch(r)
    for e in (0, 1):
        rn = (r[:, e] + 0.2).contiguous()
        a = many.propose(e, rn.repeat(Wk // few, 1).contiguous()).view(-1, few)
        b = some.propose(e, rn)
        assert torch.equal(a[0], b) and torch.equal(a[-1], b)
        assert np.isfinite(b.cpu().numpy()).all()
