"""Groups of narrow rows replay a captured graph: the calls whose schedule phase
repeats launch the graph of an earlier call instead of capturing anew (recorded on
the CPU), and each replay, with the program's own work between, is bitwise the
direct launches."""
import pytest
import torch

from gpu_util import need_gpu
from recorder import run
from workloads import configs as C

SIZES = (16, 32, 48)
STEPS = 96   # a whole number of sweeps of every member

RECORD = """
ws = []
for n in {sizes}:
    w = C.multi_system(n, n_walkers=4)
    s = P.JAGPSystem(w.system, precision=P.{precision})
    ws.append((s, P.Walkers(s, 4, adjoint=False)))
m = P.MultiSystem([k for _, k in ws])
out = []
for call in range(8):
    if call == 0 or call >= 5:   # the last three calls each after an evaluation
        for s, k in ws:
            ok(lib.qmc_eval_batch(s.h, k.h, dev(1) if call == 0 else None, None, None, None, None, None, None, None))
    r = calls(lambda: ok(lib.qmc_multi_vmc_steps(m.h, {steps}, None, None, 7, 0.3, 1, None)))
    out.append((sum(x.startswith("capture ") for x in r), sum(x.startswith("graph ") for x in r)))
"""


@pytest.mark.parametrize("precision", ["QMC_W_FP32", "QMC_MIXED", "QMC_MIXED_BF16"])
def test_calls_in_the_same_phase_replay(precision):
    out = run(RECORD.format(sizes=SIZES, steps=STEPS, precision=precision))
    assert [g for _, g in out] == [1] * 8
    # captured: the first call, the first that starts where a sweep ended, the first after
    # an evaluation; replayed: the others
    assert [c for c, _ in out] == [1, 1, 0, 0, 0, 1, 0, 0]


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["QMC_W_FP32", "QMC_MIXED", "QMC_MIXED_BF16"])
def test_replays_equal_direct_launches(precision):
    P = need_gpu()
    Wk = 8
    groups = []
    for _ in range(2):
        ws = []
        for n in SIZES:
            w = C.multi_system(n, n_walkers=Wk)
            k = P.Walkers(P.JAGPSystem(w.system, precision=getattr(P, precision)), Wk, adjoint=False)
            k.eval_batch(torch.tensor(w.r0, device="cuda"))
            ws.append(k)
        groups.append((P.MultiSystem(ws), ws))
    (mg, gw), (md, dw) = groups
    for call in range(8):
        if call >= 5:
            for k in gw + dw:
                k.eval_batch(None)
        before = [k.read(P.STATE_R) for k in gw]
        mg.vmc_steps(STEPS, seed=77, sigma=0.3, use_graph=True)
        md.vmc_steps(STEPS, seed=77, sigma=0.3, use_graph=False)
        torch.cuda.synchronize()
        for a, b, r in zip(gw, dw, before):
            assert not torch.equal(a.read(P.STATE_R), r)
            for item in (P.STATE_R, P.STATE_LOGABS, P.STATE_SIGN, P.STATE_W, P.STATE_AINV):
                assert torch.equal(a.read(item), b.read(item)), (call, item)
    mg.close(); md.close()
