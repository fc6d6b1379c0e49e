"""The per-tile gradient contractions at the sizes where their blocks can go wrong: tiles below, at and above whole
blocks of 32 rows and chunks of 8 contraction entries, tiles that begin at any column, and ranks around the units of 16
and the items of 64.

grad L = W' R^H, grad R = L^H W', grad Q = (W + W^T) conj(Q), grad Z = (W + W^T) / 2 with W = D^H (D X - U) against
complex128, entry by entry. Bound: every rounding on the way, first order (u = 2^-24): X from its factors, r and W as
sums of 2 n real products each, then the sum W' and the contraction."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24
# (tile sizes, off-diagonal rank, diagonal rank or -1)
LAYOUTS = [([1, 1], 1, 1), ([7, 9, 8], 3, 5), ([31, 33, 32], 15, 16), ([65, 40, 17], 17, 17), ([100, 64, 36], 33, -1),
           ([96, 95, 97], 48, 49), ([150, 130], 64, 65), ([140, 137], 130, 100)]


@pytest.mark.parametrize("sizes,off,diag", LAYOUTS)
def test_gradient_entry_by_entry(sizes, off, diag):
    import paper_2412_14973_amd as tl
    n, nr, ns = len(sizes), sum(sizes), 40
    start = np.concatenate([[0], np.cumsum(sizes)])
    pairs = [(i, j) for i in range(n) for j in range(i)]
    ranks = [min(off, sizes[i], sizes[j]) for i, j in pairs]
    kd = [-1 if diag < 0 else min(diag, s) for s in sizes]
    plan = tl.Plan(np.array(sizes), np.array(ranks, dtype=np.int32), np.array(kd, dtype=np.int32), ns)
    gen = torch.Generator(device="cuda").manual_seed(nr)

    def rand(*shape):
        return torch.complex(torch.randn(shape, generator=gen, device="cuda"), torch.randn(shape, generator=gen, device="cuda"))
    D, U, theta = rand(ns, nr), rand(ns, nr), rand(plan.theta_size)
    f, g = tl.grad(plan, D, U, theta, tl.FP32)

    def parts(v):   # the blocks of a theta-shaped vector: diagonals, then all L, then all R
        out, pos = [], 0
        for shape in ([(s, s if k < 0 else k) for s, k in zip(sizes, kd)] + [(sizes[i], k) for (i, j), k in zip(pairs, ranks)]
                      + [(k, sizes[j]) for (i, j), k in zip(pairs, ranks)]):
            out.append(v[pos:pos + shape[0] * shape[1]].reshape(shape))
            pos += shape[0] * shape[1]
        return out[:n], out[n:n + len(pairs)], out[n + len(pairs):]

    D2, U2 = D.to(torch.complex128), U.to(torch.complex128)
    diags, Ls, Rs = parts(theta.to(torch.complex128))
    X = torch.zeros(nr, nr, dtype=torch.complex128, device="cuda")
    EX = torch.zeros(nr, nr, dtype=torch.float64, device="cuda")

    def put(i, j, x, e):
        a, b = slice(start[i], start[i + 1]), slice(start[j], start[j + 1])
        X[a, b], EX[a, b] = x, e
    for i in range(n):
        q = diags[i]
        if kd[i] < 0:
            put(i, i, 0.5 * (q + q.T), 2 * U32 * 0.5 * (q.abs() + q.abs().T))
        else:
            put(i, i, q @ q.T.contiguous(), (2 * kd[i] + 4) * U32 * (q.abs() @ q.abs().T.contiguous()))
    for (i, j), k, L, R in zip(pairs, ranks, Ls, Rs):
        x, e = L @ R, (2 * k + 4) * U32 * (L.abs() @ R.abs())
        put(i, j, x, e)
        put(j, i, x.T, e.T)
    r = D2 @ X - U2
    Er = D2.abs() @ (EX + (2 * nr + 4) * U32 * X.abs()) + 2 * U32 * (U2.abs() + r.abs())
    W = D2.mH.contiguous() @ r
    aDH = D2.abs().T.contiguous()
    EW = aDH @ (Er + (2 * ns + 4) * U32 * r.abs())
    S, aS, ES = W + W.T, W.abs() + W.abs().T, EW + EW.T

    def check(got, want, bound, what):
        err = (got.to(torch.complex128) - want).abs()
        assert bool((err <= bound).all()), (what, float((err / bound).max()))

    gd, gL, gR = parts(g)
    for i in range(n):
        a = slice(start[i], start[i + 1])
        if kd[i] < 0:
            check(gd[i], 0.5 * S[a, a], 0.5 * (ES[a, a] + 2 * U32 * aS[a, a]), ("Z", i))
        else:
            q = diags[i]
            check(gd[i], S[a, a] @ q.conj(), (ES[a, a] + (2 * sizes[i] + 8) * U32 * aS[a, a]) @ q.abs(), ("Q", i))
    for (i, j), L, R, dL, dR in zip(pairs, Ls, Rs, gL, gR):
        a, b = slice(start[i], start[i + 1]), slice(start[j], start[j + 1])
        s, e, m = S[a, b].contiguous(), ES[a, b].contiguous(), aS[a, b].contiguous()
        check(dL, s @ R.mH.contiguous(), (e + (2 * sizes[j] + 8) * U32 * m) @ R.abs().T.contiguous(), ("L", i, j))
        check(dR, L.mH.contiguous() @ s, L.abs().T.contiguous() @ (e + (2 * sizes[i] + 8) * U32 * m), ("R", i, j))


# nr a multiple of 128, so W has no padding, and tiles that begin at an odd column and end with the last one: the pairs of
# entries that a load takes reach past the end of W's rows, and of W
@pytest.mark.parametrize("sizes,off,diag", [([1, 127], 1, 5), ([63, 65], 20, 17), ([3, 252, 1], 1, 1), ([127, 129], 40, -1)])
def test_gradient_to_the_end_of_w(sizes, off, diag):
    test_gradient_entry_by_entry(sizes, off, diag)
