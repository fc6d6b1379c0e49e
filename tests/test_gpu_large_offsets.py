"""Gradient and assembly where a matrix or a factor passes 4 GiB, which byte offsets of 32 bits do not reach: nr 23296 in
the BF16 split, whose planes of X are half as large as W = D^H r (4.3 GB). Tiles beyond the first 4 GiB of W; one tile
that W's rows leave in the middle of its contraction; a factor Q of 4.3 GB.

The factors are zero but for some rows and rank entries (the first, the last, and those around 2^31 and 2^32 bytes), so
every sum has few terms that are not zero and the bounds stay narrow. They are those of the entry-by-entry tests of the
smaller sizes: BF16 products of K terms within sqrt(2) (2^-16 + (6 K + 8) 2 u) of the sums of absolute values, FP32 sums of
2 K products within (2 K + 8) 2 u."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24
NR, NS = 23296, 32


def _bf16_bound(K):
    return 2 ** 0.5 * (2.0 ** -16 + (6 * K + 8) * 2 * U32)


def _some(n, gen):
    """Indices into n: both ends, the neighbourhoods of powers of two in bytes of rows of NR, and some at random."""
    at = {0, 1, n - 1, n - 2} | {x + q for x in (2 ** 31 // (8 * NR), 2 ** 32 // (8 * NR)) for q in (-1, 0, 1)}
    at |= set(torch.randint(0, n, (24,), generator=gen, device="cuda").tolist())
    return sorted(x for x in at if 0 <= x < n)


@pytest.mark.parametrize("sizes,off,diag", [([8192, 8192, 6912], 5, 7), ([NR], 0, 3), ([NR], 0, NR)])
def test_gradient_beyond_4_gib(sizes, off, diag):
    import paper_2412_14973_amd as tl
    n = len(sizes)
    start = np.concatenate([[0], np.cumsum(sizes)])
    pairs = [(i, j) for i in range(n) for j in range(i)]
    plan = tl.Plan(np.array(sizes), np.full(len(pairs), off, dtype=np.int32), np.full(n, diag, dtype=np.int32), NS)
    gen = torch.Generator(device="cuda").manual_seed(n + diag)

    def rand(*shape):
        return torch.complex(torch.randn(shape, generator=gen, device="cuda"), torch.randn(shape, generator=gen, device="cuda"))
    D, U = rand(NS, NR), rand(NS, NR)
    theta = torch.zeros(plan.theta_size, dtype=torch.complex64, device="cuda")

    def parts(v):   # the blocks of a theta-shaped vector: diagonals, then all L, then all R
        out, pos = [], 0
        for shape in ([(s, diag) for s in sizes] + [(sizes[i], off) for i, _ in pairs] + [(off, sizes[j]) for _, j in pairs]):
            out.append(v[pos:pos + shape[0] * shape[1]].view(shape))
            pos += shape[0] * shape[1]
        return out[:n], out[n:n + len(pairs)], out[n + len(pairs):]

    terms = 0
    for block in sum(parts(theta), []):
        rows, cols = (torch.tensor(_some(s, gen), device="cuda") for s in block.shape)
        block[rows[:, None], cols[None, :]] = rand(rows.numel(), cols.numel())
        terms = max(terms, rows.numel(), cols.numel())

    f, r, _ = tl.forward(plan, D, U, theta, tl.BF16X3, want_r=True)
    _, g = tl.grad(plan, D, U, theta, tl.BF16X3)
    wide = torch.complex128
    D2, r2 = D.to(wide), r.to(wide)
    aD, ar = D2.abs(), r2.abs()

    def cols(i):
        return slice(start[i], start[i + 1])

    def check(got, want, bound, what):
        err = (got.to(wide) - want).abs()
        assert bool((err <= bound).all()), (what, float((err / bound.clamp_min(1e-300)).max()))

    def grad_block(got, i, j, F, transposed, what):
        """(W + W^T)_ij conj(F) from W = D^H r, for F with rows in tile j; 2048 columns of F at a time."""
        Di, Dj, ri, rj = D2[:, cols(i)], D2[:, cols(j)], r2[:, cols(i)], r2[:, cols(j)]
        beta = _bf16_bound(NS) + (2 * terms + 8) * 2 * U32
        for c in range(0, F.shape[1], 2048):
            q = F[:, c:c + 2048].to(wide).conj()
            want = Di.mH.contiguous() @ (rj @ q) + ri.T.contiguous() @ (Dj.conj() @ q)
            mag = Di.abs().T.contiguous() @ (rj.abs() @ q.abs()) + ri.abs().T.contiguous() @ (Dj.abs() @ q.abs())
            part = got[c:c + 2048].T if transposed else got[:, c:c + 2048]
            check(part, want, beta * mag, what)

    # r = D X - U by factors: X_ij = A B with A, B the tile's factors, or theirs transposed above the diagonal
    Q, L, R = parts(theta)
    want = -U.to(wide)
    mag = torch.zeros(NS, NR, dtype=torch.float64, device="cuda")
    for i in range(n):
        q = Q[i][:, Q[i].abs().sum(0) > 0].to(wide)
        want[:, cols(i)] += (D2[:, cols(i)] @ q) @ q.T.contiguous()
        mag[:, cols(i)] += (aD[:, cols(i)] @ q.abs()) @ q.abs().T.contiguous()
    for (i, j), a, b in zip(pairs, L, R):
        a, b = a.to(wide), b.to(wide)
        for x, y, A, B in ((i, j, a, b), (j, i, b.T.contiguous(), a.T.contiguous())):
            want[:, cols(y)] += (D2[:, cols(x)] @ A) @ B
            mag[:, cols(y)] += (aD[:, cols(x)] @ A.abs()) @ B.abs()
    check(r, want, (_bf16_bound(n * terms) + (2 * terms + 4) * U32) * mag + 2 * U32 * (U.abs().double() + want.abs()), "r")

    gQ, gL, gR = parts(g)
    for i in range(n):
        grad_block(gQ[i], i, i, Q[i], False, ("Q", i))
    for (i, j), a, b, ga, gb in zip(pairs, L, R, gL, gR):
        grad_block(ga, i, j, b.mH.conj(), False, ("L", i, j))     # W' R^H: F = R^T
        grad_block(gb, j, i, a, True, ("R", i, j))               # (L^H W')^T = W'^T conj(L)


def test_fields_of_4_gib_are_refused():
    """A field below 4 GiB that its padding takes past it: an error from every FP32 call, not the field's first rows
    again in place of the padding."""
    import paper_2412_14973_amd as tl
    nr, ns = 1000, 536870
    plan = tl.Plan(np.array([nr]), np.zeros(0, dtype=np.int32), np.ones(1, dtype=np.int32), ns)
    D = torch.zeros(ns, nr, dtype=torch.complex64, device="cuda")
    theta = torch.zeros(plan.theta_size, dtype=torch.complex64, device="cuda")
    for call in (lambda: tl.adjoint(plan, D, D), lambda: tl.forward(plan, D, D, theta), lambda: tl.grad(plan, D, D, theta),
                 lambda: tl.forward_tlr(plan, D, D, theta), lambda: tl.solve(plan, D, D, theta, iters=1)):
        with pytest.raises(tl._lib.TLRMDDError, match="invalid argument"):
            call()
