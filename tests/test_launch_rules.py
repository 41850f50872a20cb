"""Where the faster of two kernels changes with the number of walkers (recorded,
nothing runs): each side of the lines at which both were measured."""
import inspect

import pytest

from recorder import run
from test_gpu_chain import _system

HEAD = inspect.getsource(_system)
EVAL = """
s = _system({n}, {n}, {shells}, 64)
s.L = len(s.zeta)
h = P.JAGPSystem(s)
k = P.Walkers(h, {walkers}, adjoint=False)
out = [x[0] for x in kernels(lambda: ok(lib.qmc_eval_batch(h.h, k.h, dev(1), dev(2), dev(3), dev(4), dev(5), dev(6),
                                                           dev(7), None)))]
"""


@pytest.mark.parametrize("n,shells,walkers,one", [
    (5, (0, 0, 0, 1), 65536, True), (16, (0, 0, 0, 0), 16384, True), (20, (0, 0), 4096, True), (20, (0, 0), 4097, False),
    (24, (0, 0), 512, True), (24, (0, 0), 513, False), (32, (0, 0), 16384, False), (16, (0, 0, 0, 1), 513, False)])
def test_small_systems_evaluated_in_one_launch(n, shells, walkers, one):
    out = run(HEAD + EVAL.format(n=n, shells=shells, walkers=walkers))
    assert any(x.startswith("small_eval_kernel") for x in out) == one
    assert one or any(x.startswith("dgemm_kernel") for x in out)

SR = """
import ctypes
n = lib.qmc_sr_workspace_size({samples}, {params})
out = [x[0] for x in kernels(lambda: ok(lib.qmc_sr_step({samples}, {params}, dev(1), dev(2), None, ctypes.c_double(1e-3),
    3, ctypes.c_double(0.0), dev(3), None, None, dev(4), ctypes.c_size_t(n), None)))]
"""


@pytest.mark.parametrize("samples,params,one", [(200, 168, True), (4096, 4096, True), (4096, 6000, True),
                                                (8192, 6144, False), (8192, 8192, False)])
def test_vector_work_of_a_two_pass_iteration(samples, params, one):
    out = run(SR.format(samples=samples, params=params))
    assert sum(x.startswith("sr_vec_kernel") for x in out) == (3 if one else 0)
    assert sum(x.startswith("sr_sp_kernel") for x in out) == (0 if one else 3)

PFAFFIAN = """
s = _system({n}, {n}, (0, 0, 0, 1), 64)
rng, L = np.random.default_rng(1), len(s.zeta)
s.pairing, s.pf_uu, s.pf_dd = 1, C._skew_gaussian(rng, L, 1.0 / L), C._skew_gaussian(rng, L, 1.0 / L)
s.unpaired_dn = np.zeros((L, 0))
h = P.JAGPSystem(s)
k = P.Walkers(h, 64, adjoint=False)
ok(lib.qmc_eval_batch(h.h, k.h, dev(1), None, None, None, None, None, None, None))
ok(lib.qmc_propose_move(h.h, k.h, 0, dev(1), dev(2), None, None))
out = [x for x in kernels(lambda: ok(lib.qmc_accept_move(h.h, k.h, 0, dev(1), None, None)))]
"""


@pytest.mark.parametrize("n,threads", [(2, 256), (12, 256), (13, 1024), (40, 1024)])
def test_threads_of_a_pfaffian_accept(n, threads):
    out = run(HEAD + PFAFFIAN.format(n=n))
    assert [x[2][0] for x in out if x[0].startswith("pf_accept_kernel")] == [threads]

DRIFT = """
s = _system({n}, {n}, {shells}, 64)
h = P.JAGPSystem(s, precision=P.{precision})
k = P.Walkers(h, {walkers}, adjoint=False)
ok(lib.qmc_eval_batch(h.h, k.h, dev(1), None, None, None, None, None, None, None))
out = [x[0] for x in kernels(lambda: ok(lib.qmc_propose_move(h.h, k.h, 0, dev(1), dev(2), dev(3), None)))]
"""


@pytest.mark.parametrize("n,walkers,precision,launches", [
    (10, 16384, "QMC_FP64", 1), (20, 8192, "QMC_FP64", 1), (20, 8193, "QMC_FP64", 3), (20, 16384, "QMC_MIXED", 1),
    (25, 16, "QMC_FP64", 3)])
def test_launches_of_a_proposal_with_a_drift(n, walkers, precision, launches):
    out = run(HEAD + DRIFT.format(n=n, shells=(0, 0, 0, 1), walkers=walkers, precision=precision))
    assert len(out) == launches and out[0].startswith("propose_drift_small" if launches == 1 else "propose_prep")

RUNS = """
rng = np.random.default_rng(3)
A, n = {nuclei}, {n}
center, l, m, zeta = C._shell_basis(rng, A, {shells}, 0.1, 10.0)
L = len(zeta)
s = C.System(name="wide", R=rng.uniform(0, 30.0, (A, 3)), Z=np.full(A, 2.0), center=center, l=l, m=m, zeta=zeta,
             radial=np.zeros(L, np.int32), lam=C._sym_gaussian(rng, L, 1.0 / L), n_up=n, n_dn=n, unpaired=np.zeros((L, 0)),
             j1_form=2, j1_b=np.ones(A), j2_form=1, j2=np.array([1.0, 1.0]), refresh_every=64)
h = P.JAGPSystem(s, precision=P.{precision})
k = P.Walkers(h, 2048, adjoint=False)
ok(lib.qmc_eval_batch(h.h, k.h, dev(1), None, None, None, None, None, None, None))
out = [x[0] for x in kernels(lambda: ok(lib.qmc_vmc_steps(h.h, k.h, 0, 40, dev(1), dev(2), None, None)))]
"""


@pytest.mark.parametrize("nuclei,n,shells,precision,kernel", [
    (256, 128, (0,) * 4, "QMC_FP64", "chain_kernel"), (256, 128, (0,) * 4, "QMC_REFINED", "chain_kernel"),
    (256, 1, (0,) * 4, "QMC_FP64", "chain_kernel"), (64, 40, (0, 0, 0, 1), "QMC_MIXED", "accept_prep_staged_kernel"),
    (64, 129, (0, 0, 0, 1), "QMC_FP64", "accept_prep_kernel")])
def test_fused_accepts_staged_in_lds_are_of_narrow_rows(nuclei, n, shells, precision, kernel):
    # the largest systems that could be staged have resident moves in FP64 rows
    out = run(RUNS.format(nuclei=nuclei, n=n, shells=shells, precision=precision))
    names = {"chain_kernel", "accept_prep_staged_kernel", "accept_prep_kernel"}
    assert {x for x in names if any(y.startswith(x + "I") for y in out)} == {kernel}
