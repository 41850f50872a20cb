"""QMC_FP64 proposals from the transposed rows: the padded layout at row counts
around its steps (blocked stream up to 256 rows, plain stream past them, several
chunks past 128), with and without unpaired orbitals.

What is skipped changes a ratio by at most 1e-19, so the FP64 bars hold: ratio
relative 1e-10, chain positions equal to the oracle's, log|Psi| to 1e-10.
"""
import numpy as np
import pytest
import torch

from gpu_util import need_gpu, rel_err
from oracle import jagp as O
from workloads import configs as C

pytestmark = pytest.mark.gpu


def _system(n_up, n_dn, seed=3):
    """Helium-like nuclei, enough functions for a regular W, some of them far from any electron's reach."""
    rng = np.random.default_rng(seed + 1000 * n_up + n_dn)
    N = n_up + n_dn
    A = max(2, (N + 1) // 2)
    R = C._place_nuclei(rng, A, (60.0 * N) ** (1 / 3) + 3.0)
    center, l, m, zeta = C._shell_basis(rng, A, [0, 0, 0, 1], 0.1, 10.0)
    L = len(zeta)
    return C.System(name="screened", R=R, Z=np.full(A, 2.0), center=center, l=l, m=m, zeta=zeta,
                    radial=np.zeros(L, np.int32), lam=C._sym_gaussian(rng, L, 1.0 / L), n_up=n_up, n_dn=n_dn,
                    unpaired=rng.standard_normal((L, n_up - n_dn)) / np.sqrt(L), j1_form=2, j1_b=np.ones(A),
                    j2_form=1, j2=np.array([1.0, 1.0]), refresh_every=16)


@pytest.mark.parametrize("n_up,n_dn", [(1, 1), (2, 1), (9, 9), (11, 9), (23, 23), (33, 32), (41, 41), (65, 65), (72, 70),
                                       (97, 97), (113, 113), (129, 129), (257, 255)])
def test_ratio_of_both_spins(n_up, n_dn):
    P = need_gpu()
    s = _system(n_up, n_dn)
    Wk = 3
    r = torch.tensor(C.random_positions(17, s, Wk))
    sysh = P.JAGPSystem(s)
    wk = P.Walkers(sysh, Wk, adjoint=False)
    sy = O.from_workload_system(s)
    wk.eval_batch(r.cuda())
    g = torch.Generator().manual_seed(5)
    for e in (0, n_up - 1, n_up, n_up + n_dn - 1):
        rn = r[:, e] + 0.3 * torch.randn(Wk, 3, generator=g, dtype=torch.float64)
        ratio = wk.propose(e, rn.cuda().contiguous())
        assert rel_err(ratio.cpu(), O.move_ratio(sy, r, e, rn)).max().item() <= 1e-10, e
    # the cofactor rows shared their memory with the transposed rows: an
    # evaluation restores them, and proposals after it are the same again
    a = wk.eval_batch(None)
    b = wk.eval_batch(r.cuda())
    again = wk.propose(e, rn.cuda().contiguous())
    torch.cuda.synchronize()
    assert torch.equal(a["e_loc"], b["e_loc"]) and torch.equal(a["drift"], b["drift"])
    assert torch.equal(again, ratio)


@pytest.mark.parametrize("n_up,n_dn", [(5, 4), (11, 11), (18, 17), (34, 33)])
def test_chain_equals_oracle(n_up, n_dn):
    P = need_gpu()
    s = _system(n_up, n_dn)
    Wk, steps = 4, 2 * (n_up + n_dn)
    r = torch.tensor(C.random_positions(23, s, Wk))
    disp, unif = (torch.tensor(x) for x in C.chain_arrays(29, steps, Wk))
    sysh = P.JAGPSystem(s)
    wk = P.Walkers(sysh, Wk, adjoint=False)
    wk.eval_batch(r.cuda())
    wk.vmc_steps(0, disp.cuda(), unif.cuda())
    rg, la = wk.read(P.STATE_R).cpu(), wk.read(P.STATE_LOGABS).cpu()
    sy = O.from_workload_system(s)
    rf, _, _ = O.run_chain(sy, r, disp, unif)
    assert torch.equal(rg, rf)
    assert rel_err(la, O.log_psi(sy, rf)[0]).max().item() <= 1e-10
