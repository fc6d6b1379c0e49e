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
