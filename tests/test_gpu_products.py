"""Dense FP32 products at the sizes where their tiling can go wrong: below, at and above whole blocks (32),
tiles (64, 128) and chunks of k (8, 16), contraction split over waves and not, the wide store tiles.

r = D X - U and X_adj = D^H U against complex128 products of the same complex64 operands, entry by entry. Bound: a
sum of 2 K real products in any order is within gamma_(2 K + 2) = (2 K + 4) u of sum |a||b| (u = 2^-24), four times
that in the three-product form, whose intermediate sums reach 2 |a||b|."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24
# (nr, ns): the split contraction up to 8191 blocks of 32 x 32; (4096, 256): its adjoint product in wide tiles
SIZES = [(1, 1), (7, 40), (31, 33), (32, 32), (33, 31), (64, 63), (65, 129), (127, 160), (130, 16), (257, 95), (2912, 40),
         (4096, 256)]


@pytest.mark.parametrize("form", ["FP32", "FP32_3M"])
@pytest.mark.parametrize("nr,ns", SIZES)
def test_products_entry_by_entry(nr, ns, form):
    import paper_2412_14973_amd as tl
    d = min(nr, 128)
    tiles = [d] * (nr // d) + ([nr % d] if nr % d else [])
    n = len(tiles)
    plan = tl.Plan(np.array(tiles), np.ones(n * (n - 1) // 2, dtype=np.int32), np.ones(n, dtype=np.int32), ns)
    gen = torch.Generator(device="cuda").manual_seed(100 * nr + ns)

    def rand(*shape):
        return torch.complex(torch.randn(shape, generator=gen, device="cuda"), torch.randn(shape, generator=gen, device="cuda"))
    D, U, theta = rand(ns, nr), rand(ns, nr), rand(plan.theta_size)
    c = 4.0 if form == "FP32_3M" else 1.0
    prec = getattr(tl, form)

    f, r, X = tl.forward(plan, D, U, theta, prec, want_r=True, want_X=True)
    D2, U2, X2 = (t.to(torch.complex128) for t in (D, U, X))
    ref = D2 @ X2 - U2
    bound = c * (2 * nr + 4) * U32 * (D2.abs() @ X2.abs()) + 2 * U32 * (U2.abs() + ref.abs())
    err = (r.to(torch.complex128) - ref).abs()
    assert bool((err <= bound).all()), float((err / bound).max())
    # f: FP32 sums over the 16 rows of a lane (32 roundings), FP64 from there on
    fr = 0.5 * float(torch.view_as_real(r).double().square().sum())
    assert abs(float(f) - fr) <= 34 * U32 * fr

    W = tl.adjoint(plan, D, U, prec)
    ref = D2.mH.contiguous() @ U2
    bound = c * (2 * ns + 4) * U32 * (D2.abs().T.contiguous() @ U2.abs())
    err = (W.to(torch.complex128) - ref).abs()
    assert bool((err <= bound).all()), float((err / bound).max())


# BF16 hi+lo split: hi is within 2^-9 |x| of x and lo within 2^-18 |x| of the rest, so a product misses at most
# 3 * 2^-18 |a||b| (lo lo dropped, two roundings of lo), rounded up to 2^-16; the 6 K products of an entry are added
# in FP32, at most one unit in the last place (2 u) each. sqrt(2) from the parts to the complex entry.
def _bf16_bound(K):
    return 2 ** 0.5 * (2.0 ** -16 + (6 * K + 8) * 2 * U32)


@pytest.mark.parametrize("nr,ns", [(1, 1), (7, 40), (31, 33), (33, 31), (64, 63), (65, 129), (130, 16), (257, 95),
                                   (1000, 999), (2912, 40)])
def test_bf16_products_entry_by_entry(nr, ns):
    """One X = Q Q^T: r, W = D^H U and the gradient (W + W^T) conj(Q) with W = D^H r, whose r^T is written with r."""
    import paper_2412_14973_amd as tl
    plan = tl.Plan(np.array([nr]), np.zeros(0, dtype=np.int32), np.ones(1, dtype=np.int32), ns)
    gen = torch.Generator(device="cuda").manual_seed(100 * nr + ns)

    def rand(*shape):
        return torch.complex(torch.randn(shape, generator=gen, device="cuda"), torch.randn(shape, generator=gen, device="cuda"))
    D, U, theta = rand(ns, nr), rand(ns, nr), rand(plan.theta_size)
    f, r, X = tl.forward(plan, D, U, theta, tl.BF16X3, want_r=True, want_X=True)
    D2, U2, X2, r2 = (t.to(torch.complex128) for t in (D, U, X, r))
    aDH = D2.abs().T.contiguous()
    ref = D2 @ X2 - U2
    bound = (_bf16_bound(nr) + 4 * U32) * (D2.abs() @ X2.abs()) + 2 * U32 * (U2.abs() + ref.abs())
    err = (r2 - ref).abs()
    assert bool((err <= bound).all()), float((err / bound).max())

    W = tl.adjoint(plan, D, U, tl.BF16X3)
    err = (W.to(torch.complex128) - D2.mH.contiguous() @ U2).abs()
    bound = _bf16_bound(ns) * (aDH @ U2.abs())
    assert bool((err <= bound).all()), float((err / bound).max())

    fg, g = tl.grad(plan, D, U, theta, tl.BF16X3)
    assert float(fg) == float(f)
    Q = theta.to(torch.complex128).reshape(nr, -1)
    W2 = D2.mH.contiguous() @ r2
    G = (W2 + W2.T) @ Q.conj()
    bW = _bf16_bound(ns) * (aDH @ r2.abs())
    bound = (bW + bW.T) @ Q.abs() + (2 * nr + 8) * 2 * U32 * ((W2.abs() + W2.abs().T) @ Q.abs())
    err = (g.to(torch.complex128).reshape(nr, -1) - G).abs()
    assert bool((err <= bound).all()), float((err / bound).max())


# one block per wave alone, two by two in the batch (BF16: from 256 tiles of 64 x 64 on, here 56 a problem; three
# FP32 products: from 2048 workgroups on, here 128 a problem for [a | b])
@pytest.mark.parametrize("form,count", [("BF16X3", 8), ("FP32_3M", 33), ("FP32", 33)])
def test_tiles_agree_bit_for_bit(form, count):
    """A wave's tile (one block of 32 x 32, or two by two) follows the launch; the sums do not."""
    import paper_2412_14973_amd as tl
    nr, ns = 450, 420
    prec = getattr(tl, form)
    plans = [tl.Plan(np.array([150, 150, 150]), np.full(3, 4, dtype=np.int32), np.full(3, 5, dtype=np.int32), ns)
             for _ in range(count)]
    gen = torch.Generator(device="cuda").manual_seed(3)

    def rand(*shape):
        return torch.complex(torch.randn(shape, generator=gen, device="cuda"), torch.randn(shape, generator=gen, device="cuda"))
    D, U = ([rand(ns, nr) for _ in range(count)] for _ in range(2))
    th = [0.1 * rand(plans[0].theta_size) for _ in range(count)]
    thb, fb = tl.solve_batched(plans, D, U, th, iters=4, precision=prec, resid_refresh=2)
    for i in range(0, count, 7):
        t1, f1 = tl.solve(plans[i], D[i], U[i], th[i], iters=4, precision=prec, resid_refresh=2)
        assert torch.equal(t1, thb[i]) and torch.equal(f1, fb[i])


def test_bf16_unsplit_solve():
    """Above 8191 blocks a wave contracts alone: the line products against the FP32 solve (tolerance of the mode)."""
    import paper_2412_14973_amd as tl
    nr, ns = 2912, 40
    plan = tl.Plan(np.array([1456, 1456]), np.full(1, 3, dtype=np.int32), np.full(2, 3, dtype=np.int32), ns)
    gen = torch.Generator(device="cuda").manual_seed(4)

    def rand(*shape):
        return torch.complex(torch.randn(shape, generator=gen, device="cuda"), torch.randn(shape, generator=gen, device="cuda"))
    D, U, th = rand(ns, nr) / ns, rand(ns, nr), rand(plan.theta_size)
    out = [tl.solve(plan, D, U, th, iters=3, precision=p) for p in (tl.FP32, tl.BF16X3)]
    (t0, f0), (t1, f1) = out
    assert float(((f0 - f1).abs() / f0).max()) <= 5e-3
    assert float((t0 - t1).norm() / t0.norm()) <= 5e-3


# the contraction split over waves, and (above 8191 blocks) not
@pytest.mark.parametrize("nr,ns", [(96, 70), (2912, 2912)])
@pytest.mark.parametrize("form", ["FP32", "FP32_3M", "BF16X3"])
def test_objective_sums_of_few_products(nr, ns, form):
    """theta = 0, so r = -U exactly, with |Re u|^2 = 1 and |Im u|^2 = 2^-26. A lane's FP32 sums hold one component of 16
    rows at most: 16 and 16 2^-26 are exact there, and the FP64 additions from there on, under 2^10 in a row, err by
    2^10 2^-53 = 1.2e-13 at the most. With both components in one FP32 sum the small ones vanish, 1.5e-8 of f."""
    import paper_2412_14973_amd as tl
    plan = tl.Plan(np.array([nr]), np.zeros(0, dtype=np.int32), np.ones(1, dtype=np.int32), ns)
    D = torch.ones(ns, nr, dtype=torch.complex64, device="cuda")
    U = torch.full((ns, nr), complex(1.0, 2.0 ** -13), dtype=torch.complex64, device="cuda")
    theta = torch.zeros(plan.theta_size, dtype=torch.complex64, device="cuda")
    want = 0.5 * ns * nr * (1 + 2.0 ** -26)
    tol = 1.2e-13 * want
    f, r, _ = tl.forward(plan, D, U, theta, getattr(tl, form), want_r=True)
    assert torch.equal(r, -U) and abs(float(f) - want) <= tol
    if form == "FP32":   # the tile low-rank product's second stage, never split
        f, r = tl.forward_tlr(plan, D, U, theta, want_r=True)
        assert torch.equal(r, -U) and abs(float(f) - want) <= tol
