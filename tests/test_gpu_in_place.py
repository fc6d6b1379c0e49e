"""D and U read where the caller has them, r and the adjoint image written there: against the padded copies.

A D whose rows do not begin at 16 bytes is copied first, so the same numbers at an address 8 bytes on take the other
route: the results are the same bit for bit, whatever the workspace held before. Results that lie over an input come
out as if they did not."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _setup(tl, sizes, ns, seed):
    n, nr = len(sizes), sum(sizes)
    plan = tl.Plan(np.array(sizes), np.ones(n * (n - 1) // 2, dtype=np.int32),
                   np.array([-1] + [1] * (n - 1), dtype=np.int32), ns)
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def rand(*shape):
        return torch.complex(torch.randn(shape, generator=gen, device="cuda"), torch.randn(shape, generator=gen, device="cuda"))
    return plan, rand(ns, nr), rand(ns, nr), rand(plan.theta_size)


def _shifted(t):
    flat = torch.empty(t.numel() + 2, dtype=t.dtype, device=t.device)
    off = 1 + (flat.data_ptr() // 8) % 2
    out = flat[off:off + t.numel()].view(t.shape)
    assert out.data_ptr() % 16 == 8
    return out.copy_(t)


def _dirty(n):   # a workspace of NaN
    return torch.full((n // 8 + 8,), float("nan"), dtype=torch.float64, device="cuda").view(torch.uint8)


# nr a whole number of k steps or not, one block row or more, ns below and above a block
SHAPES = [([16], 3), ([16, 32], 40), ([64], 64), ([48, 64, 32], 129), ([128, 128], 128), ([100, 44], 65), ([33], 31)]


@pytest.mark.parametrize("sizes,ns", SHAPES)
@pytest.mark.parametrize("form", ["FP32", "FP32_3M", "BF16X3"])
def test_in_place_equals_staged(sizes, ns, form):
    import paper_2412_14973_amd as tl
    prec = getattr(tl, form)
    plan, D, U, theta = _setup(tl, sizes, ns, 7 * sum(sizes) + ns)
    Ds, Us = _shifted(D), _shifted(U)
    wf, wg = _dirty(plan.workspace_bytes(tl._lib.OP_FORWARD)), _dirty(plan.workspace_bytes(tl._lib.OP_GRAD))
    f0, r0, X0 = tl.forward(plan, D, U, theta, prec, want_r=True, want_X=True, workspace=wf)
    f1, r1, X1 = tl.forward(plan, Ds, Us, theta, prec, want_r=True, want_X=True, workspace=wf)
    f2, _, _ = tl.forward(plan, D, U, theta, prec, workspace=wf)
    assert torch.equal(r0, r1) and torch.equal(X0, X1) and float(f0) == float(f1) == float(f2)
    assert bool(torch.isfinite(torch.view_as_real(r0)).all())
    (fa, ga), (fb, gb) = tl.grad(plan, D, U, theta, prec, workspace=wg), tl.grad(plan, Ds, Us, theta, prec, workspace=wg)
    assert torch.equal(ga, gb) and float(fa) == float(fb) == float(f0)
    assert torch.equal(tl.adjoint(plan, D, U, prec, workspace=wg), tl.adjoint(plan, Ds, Us, prec, workspace=wg))
    if form == "FP32":
        wt = _dirty(tl.tlr_workspace_bytes(plan))
        ft, rt = tl.forward_tlr(plan, D, U, theta, want_r=True, workspace=wt)
        fs, rs = tl.forward_tlr(plan, Ds, Us, theta, want_r=True, workspace=wt)
        fn, _ = tl.forward_tlr(plan, D, U, theta, want_r=False, workspace=wt)
        assert torch.equal(rt, rs) and float(ft) == float(fs) == float(fn)
        assert float((rt - r0).norm() / r0.norm()) <= 1e-5


def _p(t):
    return ctypes.c_void_p(t.data_ptr())


@pytest.mark.parametrize("sizes,ns", [([48, 64, 32], 129), ([128, 128], 128), ([100, 44], 65)])
def test_results_over_inputs(sizes, ns):
    """C interface: r over U, over D and one row into U; the adjoint image over D."""
    import paper_2412_14973_amd as tl
    lib = tl._lib.load()
    plan, D, U, theta = _setup(tl, sizes, ns, 5)
    nr = sum(sizes)
    f = torch.empty((), dtype=torch.float64, device="cuda")
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    ws = torch.empty(max(plan.workspace_bytes(tl._lib.OP_GRAD), tl.tlr_workspace_bytes(plan)), dtype=torch.uint8, device="cuda")

    def forward(d, u, r):
        tl._lib.check(lib.tlrmdd_forward(plan.handle, _p(d), _p(u), _p(theta), _p(f), _p(r), None, tl.FP32, _p(ws),
                                         ws.numel(), stream), "forward")

    def forward_tlr(d, u, r):
        tl._lib.check(lib.tlrmdd_forward_tlr(plan.handle, _p(d), _p(u), _p(theta), _p(f), _p(r), _p(ws), ws.numel(),
                                             stream), "forward_tlr")
    for call in (forward, forward_tlr):
        want = torch.empty_like(U)
        call(D, U, want)
        over = U.clone()
        call(D, over, over)
        assert torch.equal(over, want)
        over = D.clone()
        call(over, U, over)
        assert torch.equal(over, want)
        room = torch.zeros(ns + 2, nr, dtype=U.dtype, device="cuda")
        room[1:-1] = U
        call(D, room[1:-1], room[:-2])
        assert torch.equal(room[:-2], want)
    want = tl.adjoint(plan, D, U)
    room = torch.zeros(max(ns, nr), nr, dtype=D.dtype, device="cuda")
    room[:ns] = D
    tl._lib.check(lib.tlrmdd_adjoint(plan.handle, _p(room), _p(U), _p(room), tl.FP32, _p(ws), ws.numel(), stream), "adjoint")
    assert torch.equal(room[:nr], want)
