"""The resident chain (a run of moves of a small system in one launch): row
counts around its thread layouts (8, 16, 32 lanes a row; the rows of a matrix
tile), one and two basis functions a thread, unpaired orbitals, a Jastrow basis,
refresh periods, runs that end and start anywhere in a sweep, and the hand-over
to and from the per-move calls.

Bars as for every FP64 chain: positions and accept counts equal to the oracle's,
log|Psi| to 1e-10 relative, W^{-1} to 1e-9 of its largest entry.
"""
import numpy as np
import pytest
import torch

from gpu_util import need_gpu, rel_err
from oracle import jagp as O
from workloads import configs as C

pytestmark = pytest.mark.gpu


def _system(n_up, n_dn, shells=(0, 0, 0, 1), every=16, jastrow=False, seed=7):
    rng = np.random.default_rng(seed + 1000 * n_up + n_dn)
    N = n_up + n_dn
    A = max(2, (N + 1) // 2)
    R = C._place_nuclei(rng, A, (60.0 * N) ** (1 / 3) + 3.0)
    center, l, m, zeta = C._shell_basis(rng, A, list(shells), 0.1, 10.0)
    L = len(zeta)
    s = C.System(name="chain", R=R, Z=np.full(A, 2.0), center=center, l=l, m=m, zeta=zeta,
                 radial=np.zeros(L, np.int32), lam=C._sym_gaussian(rng, L, 1.0 / L), n_up=n_up, n_dn=n_dn,
                 unpaired=rng.standard_normal((L, n_up - n_dn)) / np.sqrt(L), j1_form=2, j1_b=np.ones(A),
                 j2_form=1, j2=np.array([1.0, 1.0]), refresh_every=every)
    return C.add_jastrow_basis(s, rng, shells=((0, 0), (1, 0))) if jastrow else s


def _setup(P, s, Wk, seed=31, precision=None):
    r = torch.tensor(C.random_positions(seed, s, Wk))
    sysh = P.JAGPSystem(s, precision=P.QMC_FP64 if precision is None else precision)
    wk = P.Walkers(sysh, Wk, adjoint=False)
    wk.eval_batch(r.cuda())
    return wk, r


@pytest.mark.parametrize("n_up,n_dn,shells,every,jastrow", [
    (1, 1, (0, 0, 1), 32, False), (2, 0, (0, 0, 1), 32, True), (4, 4, (0, 0, 0, 1), 1, False), (8, 7, (0, 0, 0, 1), 32, True),
    (9, 9, (0, 0, 0, 1), 5, False), (16, 16, (0, 0, 0, 1), 64, False), (17, 15, (0, 0, 1), 16, True),
    (20, 20, (0, 0, 0, 0, 1, 1, 2), 32, False), (33, 31, (0, 1), 32, False), (33, 33, (0, 0, 0, 1), 8, True),
    (5, 4, (0, 0, 0, 0, 0, 0, 0, 1, 1, 1, 1, 1, 1, 2, 2, 2, 2, 2, 2, 2, 2), 5, False)])
def test_chain_equals_oracle(n_up, n_dn, shells, every, jastrow):
    P = need_gpu()
    s = _system(n_up, n_dn, shells, every, jastrow)
    N, Wk = n_up + n_dn, 3
    steps, e0 = max(70, N + N // 2) if N < 40 else N + 9, N // 3   # past 64 steps, from the middle of a spin
    disp, unif = (torch.tensor(x) for x in C.chain_arrays(37, steps, Wk))
    wk, r = _setup(P, s, Wk)
    cnt = torch.full((Wk,), 5, dtype=torch.int32, device="cuda")
    wk.vmc_steps(e0, disp.cuda(), unif.cuda(), cnt)
    rg, la, sg = wk.read(P.STATE_R).cpu(), wk.read(P.STATE_LOGABS).cpu(), wk.read(P.STATE_SIGN).cpu()
    W, A = wk.read(P.STATE_W).cpu(), wk.read(P.STATE_AINV).cpu()
    sy = O.from_workload_system(s)
    rf, _, acc = O.run_chain(sy, r, disp, unif, e_start=e0)
    assert torch.equal(rg, rf)
    assert torch.equal(cnt.cpu(), 5 + acc.sum(0).to(torch.int32))
    ref = O.evaluate(sy, rf, with_intermediates=True)
    assert rel_err(la, ref["logabs"]).max().item() <= 1e-10
    assert torch.equal(sg, ref["sign"])
    assert ((W - ref["W"]).abs().max() / ref["W"].abs().max()).item() <= 1e-12
    assert ((A - ref["A"]).abs().amax((1, 2)) / ref["A"].abs().amax((1, 2))).max().item() <= 1e-9
    # the evaluation at the chain's positions reuses the P rows that the chain built
    out = wk.eval_batch(None)
    assert rel_err(out["e_loc"].cpu(), ref["e_loc"]).max().item() <= 1e-10


@pytest.mark.parametrize("precision,jastrow", [("QMC_FP64", True), ("QMC_REFINED", False)])
def test_calls_of_any_length_and_single_moves(precision, jastrow):
    # one call, calls of uneven lengths (bitwise the same), and calls with
    # propose / accept moves of the same draws in between
    P = need_gpu()
    s = _system(11, 9, jastrow=jastrow)
    Wk, steps, N = 5, 150, 20
    disp, unif = (torch.tensor(x).cuda() for x in C.chain_arrays(41, steps, Wk))
    res = []
    for sizes in ([steps], [1, 2, 7, 13, 66, 61], [3, -4, 10, -1, 30, -9, 93]):
        wk, r = _setup(P, s, Wk, precision=getattr(P, precision))
        t = 0
        for m in sizes:
            if m > 0:
                wk.vmc_steps(t % N, disp[t:t + m].contiguous(), unif[t:t + m].contiguous())
            for k in range(-m):
                e = (t + k) % N
                q = wk.propose(e, (wk.read(P.STATE_R)[:, e] + disp[t + k]).contiguous())
                wk.accept(e, (unif[t + k] < q * q).to(torch.uint8))
            t += abs(m)
        assert t == steps
        res.append([wk.read(k).cpu() for k in (P.STATE_R, P.STATE_LOGABS, P.STATE_AINV, P.STATE_W)])
    for x, y in zip(res[0], res[1]):
        assert torch.equal(x, y)
    assert torch.equal(res[0][0], res[2][0])
    assert rel_err(res[2][1], res[0][1]).max().item() <= 1e-10
    sy = O.from_workload_system(s)
    rf, _, _ = O.run_chain(sy, r, disp.cpu(), unif.cpu())
    assert torch.equal(res[0][0], rf)


@pytest.mark.parametrize("n", [30, 64, 65])
def test_chain_with_a_wide_jastrow_basis(n):
    # 120, 256 (the most a workgroup takes) and 260 Jastrow basis functions: ratios
    # and log|Psi| against evaluations, which do not use the moving Jastrow state
    P = need_gpu()
    s = _system(n, n, (0, 0, 0, 1), 16, True)
    N, Wk, steps = 2 * n, 3, 60
    disp, unif = (torch.tensor(x).cuda() for x in C.chain_arrays(39, steps, Wk))
    wk, r = _setup(P, s, Wk)
    fresh = P.Walkers(P.JAGPSystem(s), Wk, adjoint=False)
    e0 = n - 30   # over the change of spin
    t = 0
    for m in (5, -4, 30, -3, 18):
        if m > 0:
            wk.vmc_steps((e0 + t) % N, disp[t:t + m].contiguous(), unif[t:t + m].contiguous())
        for k in range(t, t - min(m, 0)):
            e, before = (e0 + k) % N, wk.read(P.STATE_R).cuda()
            after = before.clone()
            after[:, e] += disp[k]
            a, b = fresh.eval_batch(before), fresh.eval_batch(after)
            q = wk.propose(e, after[:, e].contiguous())
            want = b["sign"] * a["sign"] * torch.exp(b["logabs"] - a["logabs"])
            assert rel_err(q.cpu(), want.cpu()).max().item() <= 1e-9
            wk.accept(e, (unif[k] < q * q).to(torch.uint8))
        t += abs(m)
        out = fresh.eval_batch(wk.read(P.STATE_R).cuda())
        assert rel_err(wk.read(P.STATE_LOGABS).cpu(), out["logabs"].cpu()).max().item() <= 1e-10
        assert torch.equal(wk.read(P.STATE_SIGN).cpu(), out["sign"].cpu())
    assert t == steps and not torch.equal(wk.read(P.STATE_R).cpu(), r)


@pytest.mark.parametrize("n", [40, 70])
def test_kept_count_of_a_run_is_the_last_proposals(n):
    P = need_gpu()
    s = _system(n, n, (0, 0, 0, 1, 1), 16)
    Wk, steps = 4, 21
    disp, unif = (torch.tensor(x).cuda() for x in C.chain_arrays(45, steps, Wk))
    a, _ = _setup(P, s, Wk, precision=P.QMC_REFINED)
    b, _ = _setup(P, s, Wk, precision=P.QMC_REFINED)
    a.vmc_steps(3, disp, unif)
    b.vmc_steps(3, disp[:-1].contiguous(), unif[:-1].contiguous())
    e = (3 + steps - 1) % (2 * n)
    b.propose(e, (b.read(P.STATE_R)[:, e] + disp[-1]).contiguous())
    assert torch.equal(a.read(P.STATE_KEPT), b.read(P.STATE_KEPT))
