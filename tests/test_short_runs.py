"""Moves of the large resident form one at a time: what a caller's own accept and a
run of one or two moves touch (recorded, nothing runs), and that they end where a
long run does, bit by bit (GPU), at row counts around the accept's tiles of 32
columns and its groups of rows, up and down."""
import inspect

import pytest
import torch

from gpu_util import need_gpu
from recorder import run
from test_gpu_chain import _system
from workloads import configs as C

HEAD = inspect.getsource(_system)
SCRIPT = """
s = _system({n}, {n}, (0, 0, 0, 1), 64)
h = P.JAGPSystem(s, precision=P.{precision})
k = P.Walkers(h, {walkers}, adjoint=False)
ok(lib.qmc_eval_batch(h.h, k.h, dev(1), dev(2), dev(3), dev(4), dev(5), dev(6), dev(7), None))
def acc():
    ok(lib.qmc_propose_move(h.h, k.h, 0, dev(1), dev(2), None, None))
    rec.rec_clear()
    ok(lib.qmc_accept_move(h.h, k.h, 0, dev(3), None, None))
out = [kernels(acc)]
for m in (1, 2, 8, 32):
    out.append(kernels(lambda: ok(lib.qmc_vmc_steps(h.h, k.h, 1, m, dev(1), dev(2), dev(3), None))))
"""


@pytest.mark.parametrize("precision", ["QMC_FP64", "QMC_REFINED"])
@pytest.mark.parametrize("n,walkers,single", [(80, 256, 1), (80, 1024, 2), (96, 1024, 4), (128, 256, 1)])
def test_single_moves_leave_the_other_columns_where_they_are(n, walkers, single, precision):
    accept, *runs = run(HEAD + SCRIPT.format(n=n, walkers=walkers, precision=precision))
    assert [k[0].startswith("chain_accept_kernel") for k in accept] == [True]
    assert accept[0][1] == [walkers * -(-n // 32), 1, 1]   # 32 columns a workgroup
    for m, r in zip((1, 2, 8, 32), runs):
        resident = sum(k[0].startswith("chain_kernelILi0") for k in r)
        assert resident == (0 if m <= single else 1), (m, r)
        if m <= single:
            assert sum(k[0].startswith("chain_accept_kernel") for k in r) == m


@pytest.mark.gpu
@pytest.mark.parametrize("n_up,n_dn,shells,jastrow,precision", [
    (1, 1, (0,) * 260, False, "QMC_FP64"), (32, 32, (0, 0, 0, 0, 0, 0, 1, 1, 1, 1), False, "QMC_FP64"),
    (33, 32, (0, 0, 0, 1), True, "QMC_FP64"), (65, 64, (0, 0, 0, 1), False, "QMC_REFINED"),
    (97, 97, (0, 0, 0, 1), False, "QMC_REFINED"), (60, 60, (0, 0, 0, 1), True, "QMC_FP64"), (103, 103, (0, 0, 1), False, "QMC_FP64"), (128, 127, (0, 0, 0, 1), False, "QMC_FP64")])
def test_single_moves_equal_a_run(n_up, n_dn, shells, jastrow, precision):
    P = need_gpu()
    s = _system(n_up, n_dn, shells, 64, jastrow)
    N, Wk, steps = n_up + n_dn, 5, 14
    e0 = (n_up - 7) % N   # over the change of spin
    r = torch.tensor(C.random_positions(61, s, Wk)).cuda()
    disp, unif = (torch.tensor(x).cuda() for x in C.chain_arrays(63, steps, Wk))
    sysh = P.JAGPSystem(s, precision=getattr(P, precision))
    res = []
    for sizes in ([steps], [1] * steps, [-steps]):
        wk = P.Walkers(sysh, Wk, adjoint=False)
        wk.eval_batch(r)
        cnt = torch.zeros(Wk, dtype=torch.int32, device="cuda")
        t = 0
        for m in sizes:
            if m > 0:
                wk.vmc_steps((e0 + t) % N, disp[t:t + m].contiguous(), unif[t:t + m].contiguous(), cnt)
            for k in range(-m):
                e = (e0 + k) % N
                q = wk.propose(e, (wk.read(P.STATE_R)[:, e] + disp[k]).contiguous())
                wk.accept(e, (unif[k] < q * q).to(torch.uint8))
                cnt += (unif[k] < q * q).to(torch.int32)
            t += abs(m)
        res.append([cnt] + [wk.read(i) for i in (P.STATE_R, P.STATE_LOGABS, P.STATE_SIGN, P.STATE_W, P.STATE_AINV,
                                                 P.STATE_PHI)])
    assert 0 < int(res[0][0].sum()) < Wk * steps
    for other in res[1:]:
        for a, b in zip(res[0], other):
            assert torch.equal(a, b)
