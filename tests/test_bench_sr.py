"""The bench prices an iteration of the SR step with the bytes its kernels read: one
pass over O at its size (recorded, nothing runs)."""
import bench
from recorder import run

SCRIPT = """
import ctypes
M, Pn = {samples}, {params}
n = lib.qmc_sr_workspace_size(M, Pn)
step = lambda its: [x[0] for x in kernels(lambda: ok(lib.qmc_sr_step(M, Pn, dev(1), dev(2), None, ctypes.c_double(1e-3),
    its, ctypes.c_double(0.0), dev(3), None, None, dev(4), ctypes.c_size_t(n), None)))]
out = [step(0), step(1)]
"""


def test_an_iteration_reads_o_once():
    M, Pn = bench.SR_SAMPLES, bench.SR_PARAMS
    none, one = run(SCRIPT.format(samples=M, params=Pn))
    more = sorted(one)
    for x in none:
        more.remove(x)
    # kernels that stream O: the fused pass, or the two products
    reads = [x for x in more if x.startswith(("sr_pass_kernel", "sr_op_kernel", "sr_colsum_kernel"))]
    assert bench.sr_iteration_bytes(M, Pn) == 8.0 * M * Pn * len(reads) == 268435456.0
