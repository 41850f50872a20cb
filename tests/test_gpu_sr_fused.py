"""The SR step's one-pass iterations (at most 8192 parameters) against the
two-pass ones (the same call with the smaller workspace) and a direct solve: one
to eight columns a thread, odd counts, fewer samples than workgroups, one
sample, an O that is not 16-byte aligned, and the column limit from both sides.

f is the same arithmetic on both paths; the step solves a system whose condition
number is at most (P + eps) / eps, so the paths agree to that times the rounding
unit times the tolerance reached.
"""
import ctypes

import pytest
import torch

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu


def _inputs(M, Pn, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    n0 = -(-Pn // 16)
    Ok = torch.randn(M, Pn, generator=g, device="cuda", dtype=torch.float64)
    Ok += torch.randn(M, n0, generator=g, device="cuda", dtype=torch.float64).repeat(1, 16)[:, :Pn]
    Ok *= torch.logspace(-1, 1, Pn, device="cuda", dtype=torch.float64)
    return Ok, -5.0 + torch.randn(M, generator=g, device="cuda", dtype=torch.float64) + 0.5 * Ok[:, 0]


def _step(lib, Ok, el, wts, eps, it, tol, nbytes):
    M, Pn = Ok.shape
    p = lambda t: None if t is None else ctypes.c_void_p(t.data_ptr())  # noqa: E731
    work = torch.full((nbytes // 8,), float("nan"), dtype=torch.float64, device="cuda")
    out = [torch.full((n,), float("nan"), dtype=torch.float64, device="cuda") for n in (Pn, Pn, 1)]
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    rc = lib.qmc_sr_step(M, Pn, p(Ok), p(el), p(wts), eps, it, tol, *map(p, out), p(work), nbytes, st)
    assert rc == 0, lib.qmc_last_error().decode()
    return out


@pytest.mark.parametrize("M,Pn,weighted", [(1, 3, False), (5, 1, False), (300, 64, True), (257, 1023, False), (511, 1025, True),
                                           (64, 2050, False), (1000, 4096, True), (700, 5001, False), (513, 8192, False),
                                           (300, 8193, False)])
def test_one_pass_equals_two_pass(M, Pn, weighted):
    P = need_gpu()
    lib = P.load()
    Ok, el = _inputs(M, Pn, 100 + Pn)
    wts = 0.5 + torch.rand(M, device="cuda", dtype=torch.float64) if weighted else None
    eps, it, tol = 1e-2, 300, 1e-13
    small = 8 * (6 * Pn + M + 3 * (-(-Pn // 256)) + 16 + 2 * min(max(-(-M // 128), 1), 64) * Pn)
    full = lib.qmc_sr_workspace_size(M, Pn)
    assert full >= small and (Pn <= 8192 or full == small)
    a = _step(lib, Ok, el, wts, eps, it, tol, full)
    b = _step(lib, Ok, el, wts, eps, it, tol, small)
    c = _step(lib, Ok, el, wts, eps, it, tol, full)
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(a, c))
    assert torch.equal(a[1], b[1])
    if M == 1:   # one sample: no variance, no force
        assert a[1].abs().max().item() == 0.0 and a[0].abs().max().item() == 0.0
        return
    n = b[0].norm()
    assert ((a[0] - b[0]).norm() / n).item() <= 1e-9
    # the residual of the returned step, with torch products
    w = torch.ones(M, device="cuda", dtype=torch.float64) if wts is None else wts
    D = Ok - (w @ Ok) / w.sum()
    r = (D.T @ (w * (D @ a[0]))) / w.sum() + eps * ((w @ (D * D)) / w.sum()) * a[0] - a[1]
    assert (r.norm() / a[1].norm()).item() <= 1e-10
    assert a[2].item() <= 1e-12


def test_iteration_counts_and_alignment():
    P = need_gpu()
    lib = P.load()
    M, Pn = 200, 300
    base = torch.empty(M * Pn + 1, dtype=torch.float64, device="cuda")
    Ok, el = _inputs(M, Pn, 9)
    odd = base[1:].view(M, Pn)   # 8-byte aligned only
    odd.copy_(Ok)
    full = lib.qmc_sr_workspace_size(M, Pn)
    for it in (0, 1, 2, 7):
        x = _step(lib, Ok, el, None, 1e-3, it, 0.0, full)
        y = _step(lib, odd, el, None, 1e-3, it, 0.0, full)
        z = _step(lib, Ok, el, None, 1e-3, it, 0.0, 8 * (6 * Pn + M + 6 + 16 + 4 * Pn))
        torch.cuda.synchronize()
        for u in (y, z):
            assert all(((p - q).abs().max() <= 1e-10 * q.abs().max()).item() for p, q in zip(u, x)), it
        if it == 0:
            assert x[0].abs().max().item() == 0.0 and x[2].item() == 1.0


@pytest.mark.parametrize("M,Pn", [(2, 2), (150, 200), (1000, 1025), (2100, 2049), (1500, 2200)])
def test_nearly_square_keeps_two_passes(M, Pn):
    # well conditioned (eps = 1); the workspace does not choose the path of these sizes
    P = need_gpu()
    lib = P.load()
    Ok, el = _inputs(M, Pn, 300 + Pn)
    small = 8 * (6 * Pn + M + 3 * (-(-Pn // 256)) + 16 + 2 * min(max(-(-M // 128), 1), 64) * Pn)
    a = _step(lib, Ok, el, None, 1.0, 200, 1e-13, small)
    b = _step(lib, Ok, el, None, 1.0, 200, 1e-13, small + 8 * 300 * Pn)
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(a, b))
    D = Ok - Ok.mean(0)
    r = (D.T @ (D @ a[0])) / M + (D * D).mean(0) * a[0] - a[1]
    assert (r.norm() / a[1].norm()).item() <= 1e-10
    assert a[2].item() <= 1e-12
