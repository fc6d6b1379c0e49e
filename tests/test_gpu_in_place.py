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


def _solve_plan(tl, sizes, ns, off, diag):
    n = len(sizes)
    return tl.Plan(np.array(sizes), np.full(n * (n - 1) // 2, off, dtype=np.int32), np.full(n, diag, dtype=np.int32), ns)


@pytest.mark.parametrize("form,line", [("FP32", "LINE_DENSE"), ("FP32_3M", "LINE_TILE_GRAD"), ("BF16X3", "LINE_TILE_GRAD")])
@pytest.mark.parametrize("sizes,ns,off,diag", [([128, 128], 128, 8, 8), ([128, 128, 128, 128], 256, 16, 16),
                                               ([128, 128, 128, 128], 200, 10, 9)])
def test_solve_in_place_equals_staged(form, line, sizes, ns, off, diag):
    """Whole tiles at 16 bytes are read where they lie; at 8 bytes on they are copied. Ranks that fill their padding
    leave nothing to clear: the workspace holds NaN before."""
    import paper_2412_14973_amd as tl
    plan = _solve_plan(tl, sizes, ns, off, diag)
    _, D, U, _ = _setup(tl, sizes, ns, 11)
    gen = torch.Generator(device="cuda").manual_seed(2)
    th = 0.2 * torch.complex(torch.randn(plan.theta_size, generator=gen, device="cuda"),
                             torch.randn(plan.theta_size, generator=gen, device="cuda"))
    kw = dict(iters=4, precision=getattr(tl, form), line_products=getattr(tl, line))
    opts = tl.make_opts(4, precision=kw["precision"], line_products=kw["line_products"])
    out = [tl.solve(plan, d, u, th, workspace=_dirty(plan.workspace_bytes(tl._lib.OP_SOLVE, opts)), **kw)
           for d, u in ((D, U), (_shifted(D), _shifted(U)))]
    assert bool(torch.isfinite(out[0][1]).all()) and float(out[0][1][-1]) < float(out[0][1][0])
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


def test_batches_above_one_launch():
    """More problems than one staging launch takes (32), of different theta sizes, against each alone."""
    import paper_2412_14973_amd as tl
    sizes, ns, count = [20, 24, 20], 50, 67
    plans = [_solve_plan(tl, sizes, ns, 1 + i % 5, -1 if i % 3 == 0 else 4) for i in range(count)]
    gen = torch.Generator(device="cuda").manual_seed(6)

    def rand(*shape):
        return torch.complex(torch.randn(shape, generator=gen, device="cuda"), torch.randn(shape, generator=gen, device="cuda"))
    D, U = ([rand(ns, sum(sizes)) for _ in range(count)] for _ in range(2))
    th = [0.2 * rand(p.theta_size) for p in plans]
    thb, fb = tl.solve_batched(plans, D, U, th, iters=3)
    for i in (0, 1, 31, 32, 33, 63, 64, 66):
        t1, f1 = tl.solve(plans[i], D[i], U[i], th[i], iters=3)
        assert torch.equal(t1, thb[i]) and torch.equal(f1, fb[i]), i
