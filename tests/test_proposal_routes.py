"""Which kernels a proposal without a drift launches (recorded, nothing runs): FP64
rows whole where the transposed copy costs more than it saves (single moves of small
systems, small sets past the resident sizes), the kept columns elsewhere."""
import inspect

import pytest

from recorder import run
from test_gpu_chain import _system

HEAD = inspect.getsource(_system)
SCRIPT = """
s = _system({n}, {n}, {shells}, 64)
h = P.JAGPSystem(s, precision=P.{precision})
k = P.Walkers(h, {walkers}, adjoint=False)
ok(lib.qmc_eval_batch(h.h, k.h, dev(1), dev(2), dev(3), dev(4), dev(5), dev(6), dev(7), None))
out = [x[0] for x in kernels(lambda: ok(lib.qmc_propose_move(h.h, k.h, 0, dev(1), dev(2), None, None)))]
"""
ROWS = ["propose_prep_kernel", "propose_rows_kernel", "propose_finalize_kernel"]
COLUMNS = ["propose_prep_kernel", "propose_screened_kernel", "propose_finalize_screened_kernel"]


@pytest.mark.parametrize("n,shells,walkers,precision,want", [
    (5, (0, 0, 1), 16, "QMC_FP64", ROWS), (20, (0, 0, 0, 1), 2048, "QMC_FP64", ROWS),
    (20, (0, 0, 0, 1), 2048, "QMC_REFINED", COLUMNS), (40, (0, 0, 0, 1), 64, "QMC_FP64", ["pt_build_kernel", "chain_kernel"]),
    (129, (0, 0, 0, 1), 32, "QMC_FP64", ROWS), (129, (0, 0, 0, 1), 72, "QMC_FP64", ["pt_build_kernel"] + COLUMNS),
    (129, (0, 0, 0, 1), 32, "QMC_REFINED", COLUMNS), (256, (0, 0, 1), 2, "QMC_FP64", ["pt_build_kernel"] + COLUMNS)])
def test_kernels_of_a_proposal(n, shells, walkers, precision, want):
    out = run(HEAD + SCRIPT.format(n=n, shells=shells, walkers=walkers, precision=precision))
    assert len(out) == len(want) and all(a.startswith(b) for a, b in zip(out, want)), out
