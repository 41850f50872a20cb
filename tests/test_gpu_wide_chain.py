"""Resident moves of systems whose state leaves room for one workgroup a compute unit
(the large form with 512 threads: past 80 KiB of LDS): runs equal single moves bit for
bit, and the state they leave is that of the oracle at the walkers' positions.  Sizes on
both sides of the line, of one and two basis functions a thread, with a Jastrow basis and
with contracted orbitals."""
import numpy as np
import pytest
import torch

from gpu_util import need_gpu
from oracle import jagp as O
from recorder import run
from test_gpu_chain import _system
from test_launch_rules import HEAD
from workloads import configs as C

SYSTEMS = {
    "80": (80, 80, (0, 0, 1), False), "86": (86, 85, (0, 0, 1), False), "97": (97, 96, (0, 0, 0, 1), True),
    "112": (112, 112, (0, 0, 0, 1), False), "128": (128, 127, (0, 0, 1), False),
    "128 spread": (128, 128, (0, 0, 0, 0, 1), False),
    "91 contracted": (91, 90, (0, 0, 0, 1), False)}

THREADS = """
s = _system({n}, {n}, (0, 0, 1), 64)
h = P.JAGPSystem(s)
k = P.Walkers(h, 16, adjoint=False)
ok(lib.qmc_eval_batch(h.h, k.h, dev(1), None, None, None, None, None, None, None))
out = [x[2][0] for x in kernels(lambda: ok(lib.qmc_vmc_steps(h.h, k.h, 0, 8, dev(2), dev(3), None, None)))
       if x[0].startswith("chain_kernel")]
"""


@pytest.mark.parametrize("n,threads", [(66, 256), (84, 256), (96, 512), (128, 512)])
def test_threads_of_a_run(n, threads):
    assert run(HEAD + THREADS.format(n=n)) == [threads]


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["QMC_FP64", "QMC_REFINED"])
@pytest.mark.parametrize("name", list(SYSTEMS))
def test_runs_equal_single_moves(name, precision):
    P = need_gpu()
    n_up, n_dn, shells, jastrow = SYSTEMS[name]
    s = _system(n_up, n_dn, shells, 16, jastrow=jastrow, seed=11)
    if name.endswith("contracted"):
        s.contraction = np.eye(len(s.zeta)) + 0.3 * np.eye(len(s.zeta), k=1)
    Wk, N, T, e0 = 5, n_up + n_dn, 40, n_up - 21   # both spins, two refreshes
    r = torch.tensor(C.random_positions(31, s, Wk))
    sysh = P.JAGPSystem(s, precision=getattr(P, precision))
    a, b = (P.Walkers(sysh, Wk, adjoint=False) for _ in range(2))
    for k in (a, b):
        k.eval_batch(r.cuda())
    g = torch.Generator().manual_seed(4)
    d = (0.3 * torch.randn(T, Wk, 3, generator=g, dtype=torch.float64)).cuda()
    u = torch.rand(T, Wk, generator=g, dtype=torch.float64).cuda()
    a.vmc_steps(e0, d, u)
    for t in range(T):
        e = (e0 + t) % N
        q = b.propose(e, (b.read(P.STATE_R)[:, e] + d[t]).contiguous())
        b.accept(e, (u[t] < q * q).to(torch.uint8))
    torch.cuda.synchronize()
    for item in (P.STATE_R, P.STATE_SIGN, P.STATE_W, P.STATE_AINV, P.STATE_LOGABS):
        assert torch.equal(a.read(item), b.read(item)), item
    rows = a.read(P.STATE_R).cpu()
    assert (rows != r).any(-1).sum() > Wk * T // 4
    ref = O.evaluate(O.from_workload_system(s), rows[:2], with_intermediates=True)
    assert torch.equal(a.read(P.STATE_SIGN)[:2].cpu(), ref["sign"])
    # log|Psi| adds the logarithms of at most 16 moves to a refresh's; W's lines are sums of
    # P rows (REFINED: within 1e-14 of the largest)
    tol = 64 * 2.0 ** (-52 if precision == "QMC_FP64" else -46) * torch.linalg.cond(ref["W"]) + 1e-10 * ref["logabs"].abs()
    assert ((a.read(P.STATE_LOGABS)[:2].cpu() - ref["logabs"]).abs() <= tol).all()
