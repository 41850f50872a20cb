"""The one-launch evaluation of a small system and the resident chain over
contracted orbitals: row counts around the matrix tiles (1, 15, 16, 17, 24
rows), unpaired orbitals, a Jastrow basis, systems at the edge of the LDS bound,
contractions with their coefficients in LDS and too many for it, a singular
walker.

Bars as for every FP64 evaluation: relative 1e-10 on log|Psi|, E_kin and E_loc,
1e-8 on the drift, 1e-9 of its largest entry on W^{-1}; chains' positions and
accept counts equal to the oracle's.
"""
import numpy as np
import pytest
import torch

from gpu_util import need_gpu, rel_err
from oracle import jagp as O
from workloads import configs as C

pytestmark = pytest.mark.gpu


def _system(n_up, n_dn, shells, jastrow=False, con=0, nuclei=None):
    rng = np.random.default_rng(17 + 1000 * n_up + n_dn)
    N = n_up + n_dn
    A = nuclei or max(2, (N + 1) // 2)
    R = C._place_nuclei(rng, A, (60.0 * N) ** (1 / 3) + 3.0)
    center, l, m, zeta = C._shell_basis(rng, A, list(shells), 0.1, 10.0)
    Lq = len(zeta)
    cm = None
    if con:   # con orbitals, each over every primitive (dense) or over those of one nucleus
        dense = con * Lq <= 4096 and con % 2 == 1
        cm = rng.standard_normal((Lq, con)) / 3.0
        if not dense:
            cm *= (center[:, None] == (np.arange(con) % A)[None, :])
    L = con or Lq
    s = C.System(name="small", R=R, Z=np.full(A, 2.0), center=center, l=l, m=m, zeta=zeta,
                 radial=np.zeros(Lq, np.int32), lam=C._sym_gaussian(rng, L, 1.0 / L), n_up=n_up, n_dn=n_dn,
                 unpaired=rng.standard_normal((L, n_up - n_dn)) / np.sqrt(L), j1_form=2, j1_b=np.ones(A),
                 j2_form=1, j2=np.array([1.0, 1.0]), refresh_every=8, contraction=cm)
    return C.add_jastrow_basis(s, rng, shells=((0, 0), (1, 0))) if jastrow else s


SYSTEMS = [
    (1, 1, (0,), False, 0, None), (2, 1, (0, 0, 1, 1), True, 0, None), (15, 15, (0, 0, 1), False, 0, None),
    (16, 16, (0, 0, 0, 1), False, 0, None), (17, 13, (0, 0, 0, 1), True, 0, None), (24, 23, (0, 0, 1), False, 0, 18),
    (24, 24, (0, 0, 1), False, 0, 18), (4, 3, (0, 0, 0, 1, 1, 1, 2, 2, 2, 2), False, 0, 8),
    (5, 4, (0, 0, 1, 2), False, 11, None), (11, 9, (0, 0, 1), True, 30, None), (3, 3, (0, 0, 0, 0, 1, 1, 2, 2), False, 8, 30),
    (16, 15, (0, 0, 0, 0, 1, 1, 2), True, 60, 20), (36, 34, (0, 0, 1, 1), False, 120, None)]


@pytest.mark.parametrize("n_up,n_dn,shells,jastrow,con,nuclei", SYSTEMS)
def test_small_evaluation_equals_oracle(n_up, n_dn, shells, jastrow, con, nuclei):
    P = need_gpu()
    s = _system(n_up, n_dn, shells, jastrow, con, nuclei)
    Wk = 5
    r = torch.tensor(C.random_positions(43, s, Wk))
    if n_up > 1:
        r[2, 1] = r[2, 0]   # two equal rows of W: a singular walker
    sysh = P.JAGPSystem(s)
    wk = P.Walkers(sysh, Wk)
    ok = [w for w in range(Wk) if n_up == 1 or w != 2]
    sy = O.from_workload_system(s)
    for call in range(2):   # at given positions, then at the walkers' own
        out = wk.eval_batch(r.cuda() if call == 0 else None)
        assert torch.equal(wk.read(P.STATE_R).cpu(), r)
        ref = O.evaluate(sy, r[ok], with_intermediates=True)
        for k in ("logabs", "e_kin", "e_loc"):
            assert rel_err(out[k].cpu()[ok], ref[k]).max().item() <= 1e-10, k
        assert torch.equal(out["sign"].cpu()[ok], ref["sign"])
        d = out["drift"].cpu()[ok]
        assert ((d - ref["drift"]).abs() / ref["drift"].abs().clamp(min=1.0)).max().item() <= 1e-8
        st = out["status"].cpu()
        assert (st[ok] == 0).all() and (n_up == 1 or st[2] != 0)
        A, W = wk.read(P.STATE_AINV).cpu()[ok], wk.read(P.STATE_W).cpu()[ok]
        assert ((W - ref["W"]).abs().max() / ref["W"].abs().max()).item() <= 1e-12
        assert ((A - ref["A"]).abs().amax((1, 2)) / ref["A"].abs().amax((1, 2))).max().item() <= 1e-9


@pytest.mark.parametrize("n_up,n_dn,shells,jastrow,con,nuclei", [x for x in SYSTEMS if x[4]] + [
    (70, 66, (0, 0, 1, 1, 2, 2), False, 300, 40), (40, 40, (0, 0, 0, 0, 1, 1, 2), False, 520, 40)])
def test_contracted_chain_equals_oracle(n_up, n_dn, shells, jastrow, con, nuclei):
    P = need_gpu()
    s = _system(n_up, n_dn, shells, jastrow, con, nuclei)
    N, Wk = n_up + n_dn, 3
    steps, e0 = N + 9, N // 3
    r = torch.tensor(C.random_positions(47, s, Wk))
    disp, unif = (torch.tensor(x) for x in C.chain_arrays(53, steps, Wk))
    sy = O.from_workload_system(s)
    rf, _, acc = O.run_chain(sy, r, disp, unif, e_start=e0)
    sysh = P.JAGPSystem(s)
    for single in (0, 5):   # a run; a run with single moves before it
        wk = P.Walkers(sysh, Wk, adjoint=False)
        wk.eval_batch(r.cuda())
        cnt = torch.zeros(Wk, dtype=torch.int32, device="cuda")
        for t in range(single):
            e = (e0 + t) % N
            q = wk.propose(e, (wk.read(P.STATE_R)[:, e] + disp[t].cuda()).contiguous())
            a = (unif[t].cuda() < q * q)
            wk.accept(e, a.to(torch.uint8))
            cnt += a.to(torch.int32)
        wk.vmc_steps((e0 + single) % N, disp[single:].cuda(), unif[single:].cuda(), cnt)
        assert torch.equal(wk.read(P.STATE_R).cpu(), rf)
        assert torch.equal(cnt.cpu(), acc.sum(0).to(torch.int32))
        ref = O.evaluate(sy, rf, with_intermediates=True)
        assert rel_err(wk.read(P.STATE_LOGABS).cpu(), ref["logabs"]).max().item() <= 1e-10
        A = wk.read(P.STATE_AINV).cpu()
        assert ((A - ref["A"]).abs().amax((1, 2)) / ref["A"].abs().amax((1, 2))).max().item() <= 1e-9
        out = wk.eval_batch(None)
        assert rel_err(out["e_loc"].cpu(), ref["e_loc"]).max().item() <= 1e-10
