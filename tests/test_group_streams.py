"""The streams of a group call (recorded, nothing runs): whatever the call enqueues
on streams of its own is ordered before the caller's later work, also when a launch
in its middle fails and the call returns an error.
"""
import pytest

from recorder import run

SCRIPT = """
CALLER = 0x77
def group(precision, every, sizes=(16, 32, 64)):
    ws = []
    for n in sizes:
        w = C.multi_system(n, n_walkers=4)
        s = P.JAGPSystem(w.system, precision=precision, refresh_every=every)
        k = P.Walkers(s, 4, adjoint=False)
        ok(lib.qmc_eval_batch(s.h, k.h, dev(1), None, None, None, None, None, None, None))
        ws.append(k)
    return P.MultiSystem(ws)
def unordered(recs, caller):
    # streams with a launch that the caller's stream is not behind at the end
    seen, events, last = {{}}, {{}}, {{}}
    for i, r in enumerate(recs):
        f = r.split()
        if f[0] == "launch":
            st = f[-1]
            seen.setdefault(st, {{}})[st] = i
            last[st] = i
        elif f[0] == "record":
            events[f[1]] = dict(seen.get(f[2], {{}}))
        elif f[0] == "wait":
            mine = seen.setdefault(f[1], {{}})
            for st, k in events.get(f[2], {{}}).items():
                mine[st] = max(mine.get(st, -1), k)
    mine = seen.get(caller, {{}})
    return [st for st, k in last.items() if mine.get(st, -1) < k]
out = []
for fail in {fails}:
    m = group(P.{precision}, 8)
    fail_at(fail)
    rec.rec_clear()
    rc = lib.qmc_multi_vmc_steps(m.h, 40, None, None, 7, 0.3, 0, vp(CALLER))
    rs = records()
    fail_at(-1)
    out.append((rc, sum(r.startswith("launch") for r in rs), unordered(rs, hex(CALLER))))
    m.close()
"""


@pytest.mark.parametrize("precision", ["QMC_FP64", "QMC_REFINED", "QMC_MIXED"])
def test_the_callers_stream_waits_for_every_launch(precision):
    out = run(SCRIPT.format(fails=[-1, 0, 1, 3, 5], precision=precision))
    assert out[0][0] == 0 and out[0][1] > 5
    for rc, launches, unordered in out:
        assert unordered == []
    for rc, launches, _ in out[1:]:
        assert rc == -3   # QMC_ERR_HIP
    assert [n for _, n, _ in out[1:]] == [0, 1, 3, 5]


SHORT = SCRIPT[:SCRIPT.index("out = []")] + """
m = group(P.QMC_FP64, 8, {sizes})
out = calls(lambda: ok(lib.qmc_multi_vmc_steps(m.h, {steps}, None, None, 7, 0.3, 0, vp(CALLER))))
out = [out, unordered(out, hex(CALLER))]
"""


@pytest.mark.parametrize("sizes,steps,streams", [((16, 32), 8, 1), ((16, 32), 9, 2), ((16,) * 4, 1, 1), ((16,) * 4, 2, 4),
                                                 ((16,) * 8, 1, 4)])
def test_short_calls_of_a_few_members_stay_on_one_stream(sizes, steps, streams):
    out, unordered = run(SHORT.format(sizes=sizes, steps=steps))
    runs = [r.split() for r in out if r.startswith("launch") and "chain_kernel" in r]
    assert unordered == [] and len({r[-1] for r in runs}) == streams
    # one launch of draws, and nothing copied from the host
    assert sum("philox" in r for r in out) == 1 and not any(r.startswith("copy") for r in out)
